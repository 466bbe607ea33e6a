// GEMM and LM head for every shape and type the bf16 MFMA GEMM does not take: fp32 operands, bf16 widths that do not fill
// its 64-wide K tiles.  fp32 operands run on v_mfma_f32_16x16x4_f32 (fp32 products, fp32 sums: the arithmetic of a chain of
// fused multiply-adds), bf16 operands on v_mfma_f32_16x16x32_bf16.
//
// What bounds these shapes: with the 16 - 128 rows of a few states, the lines that a CU's L1 hands out; with several hundred
// rows the fp32 matrix pipes (256 flop per clock and CU).  Eight wavefronts share one output tile and split K (chunk c of 128
// bytes, a whole line of each row, goes to wavefront c % 8), which puts eight times as many loads in flight per tile;
// their sums are added through LDS as a fixed tree.  The K order of an element depends on K alone, not on the tile or
// on M, so a row's result does not depend on the rows computed with it.
//
// A 16x16 fragment of either type is one 16-byte load per lane whose four lane groups read 64 contiguous bytes of a row; loaded
// so, straight into registers, half lines of sixteen rows an instruction, a CU gets 14 bytes a clock.  Each wavefront
// therefore brings its chunk global -> LDS as whole lines (eight rows an instruction) into LDS of its own and reads the
// fragments there (all but the fp32 tiles of 64 x 64).  Measured, registers -> LDS, us: fp32, 64 rows, QKV 1536 x 1024 8.5 -> 6.2, gate/up 2816 x 1024 18.4 -> 15.7,
// down 1024 x 2816 17.8 -> 9.8; bf16, 128 rows, 8.4 -> 5.6, 13.8 -> 10.1, 17.3 -> 9.1.  (A kernel on vector FMAs with scalar loads
// took 200 - 340 us for these.)
#include <type_traits>

#include "kernels.h"

namespace spiffy {

namespace {

constexpr int NW = 8;                 // wavefronts of a workgroup = K slices of a tile
constexpr int RSTRIDE = 64 * 4 + 16;  // floats of one reduced 16x16 fragment in LDS (padded: see the head's transposed reads)

template <typename T> struct Frag;
template <> struct Frag<float> {
  typedef f32x4 type;
  static constexpr int KC = 16, VEC = 4;      // K values of a fragment, of one lane
};
template <> struct Frag<bf16_t> {
  typedef bf16x8 type;
  static constexpr int KC = 32, VEC = 8;
};
__device__ __forceinline__ f32x4 mma(f32x4 c, f32x4 a, f32x4 b) {
#pragma unroll
  for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
  return c;
}
__device__ __forceinline__ f32x4 mma(f32x4 c, bf16x8 a, bf16x8 b) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// LDS of one wavefront: a chunk of 128 bytes of TM * 16 activation rows and TN * 16 weight rows
constexpr int stage_bytes(int tm, int tn) { return (tm + tn) * 2048; }

__device__ __forceinline__ void wait_vmcnt0() {    // lgkmcnt / expcnt untouched
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::: "memory");                   // no LDS read moves above it
}
__device__ __forceinline__ void wait_lgkm0() {     // vmcnt / expcnt untouched
  __builtin_amdgcn_s_waitcnt(0xC07F);
  asm volatile("" ::: "memory");
}

// Sources of a wavefront's transfers.  One transfer brings a chunk of eight rows as whole 128-byte lines, global -> LDS: lane
// -> row 8 * q + lane / 8 and the 16 bytes that belong at LDS position lane % 8; position p of row r holds piece
// p ^ (r / 2) % 8, so that the reads of one piece of sixteen rows are free of bank conflicts.  Transfers 0 .. 2*TM-1 are
// activation rows, the rest weight rows; `row(i)` is the start of row i of the tile's TM*16 + TN*16.
template <typename T, int TM, int TN, typename RowFn>
__device__ __forceinline__ void tile_sources(const T* (&src)[2 * (TM + TN)], int lane, RowFn row) {
#pragma unroll
  for (int q = 0; q < 2 * (TM + TN); ++q) src[q] = row(8 * q + (lane >> 3));
}

// One output tile.  On return wavefront 0's .. 7's sums are in acc; the caller reduces them.  `stage` is this wavefront's LDS:
// nobody else reads or writes it, so the loop has no barrier.  One chunk is in flight per wavefront, the next is asked for
// as soon as the fragments are in registers; a second stage gained nothing, the workgroups it keeps off the compute unit
// cost more (fp32, 64 rows, K = 2816: 9.7 us with one stage, 11.4 with two).
template <typename T, int TM, int TN>
__device__ __forceinline__ void tile_product(const T* const (&src)[2 * (TM + TN)], int K, int wave, int lane, unsigned stage,
                                             f32x4 (&acc)[TM][TN]) {
  typedef typename Frag<T>::type frag_t;
  typedef const __attribute__((address_space(3))) frag_t* lds_frag_ptr;
  constexpr int KC = Frag<T>::KC, VEC = Frag<T>::VEC, L = 2 * (TM + TN);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // chunks of this wavefront; the last one of K may be cut short.  Every branch is wavefront-uniform.
  const int whole = K / (2 * KC), n_whole = whole > wave ? (whole - wave + NW - 1) / NW : 0;
  const bool cut = whole * 2 * KC < K && whole % NW == wave;
  const int n = n_whole + (cut ? 1 : 0);
  auto load = [&](int t) {                         // this wavefront's t-th chunk
    const int k0 = (wave + t * NW) * 2 * KC;
#pragma unroll
    for (int q = 0; q < L; ++q) {
      int k = k0 + (((lane & 7) ^ (4 * (q & 1) + (lane >> 4))) * VEC);
      if (k0 + 2 * KC > K) k = min(k, K - VEC);    // (zeroed when it is read)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   :: "s"(stage + q * 1024), "v"(src[q] + k) : "memory");
    }
  };
  const int l16 = lane & 15, g = lane >> 4, swz = (l16 >> 1) & 7;
  if (n > 0) load(0);
  for (int t = 0; t < n; ++t) {
    wait_vmcnt0();
    const unsigned base = stage + l16 * 128;
    frag_t fa[2][TM], fw[2][TN];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned p = base + (((h * 4 + g) ^ swz) * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j) fw[h][j] = *(lds_frag_ptr)(size_t)(p + (TM + j) * 2048);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[h][i] = *(lds_frag_ptr)(size_t)(p + i * 2048);
    }
    wait_lgkm0();                                  // the fragments are in registers: the stage is free
    if (t + 1 < n) load(t + 1);
    if (cut && t == n - 1) {      // K is a multiple of 8, so a lane's values are all inside K or all beyond it
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if ((2 * whole + h) * KC + g * VEC >= K) {
#pragma unroll
          for (int j = 0; j < TN; ++j) fw[h][j] = frag_t{};
#pragma unroll
          for (int i = 0; i < TM; ++i) fa[h][i] = frag_t{};
        }
    }
    // fp32: a chunk's products are summed on their own and then added, so that the long sum along K is rounded once a chunk
    // and wavefront (a layer of width 1024 against 64 bits: 5.0e-7 with one chain, 3.0e-7 so; no measurable time)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (std::is_same<T, float>::value) {
          f32x4 c = mma(f32x4{0.f, 0.f, 0.f, 0.f}, fa[0][i], fw[0][j]);
          c = mma(c, fa[1][i], fw[1][j]);
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] += c[v];
        } else {
          acc[i][j] = mma(acc[i][j], fa[0][i], fw[0][j]);
          acc[i][j] = mma(acc[i][j], fa[1][i], fw[1][j]);
        }
      }
  }
}

// The same sums in the same order with the fragments loaded straight into registers, one chunk at a time: `arow` and `wrow` are
// the lane's rows.  For the fp32 tiles of 64 x 64 (launch_epi says where): one workgroup a CU either way, and without the trip
// through LDS 1024 rows of 4104 columns, K = 1032, take 118 us instead of 129.
template <typename T, int TM, int TN>
__device__ __forceinline__ void tile_product_regs(const T* const (&arow)[TM], const T* const (&wrow)[TN], int K, int wave, int lane,
                                                  f32x4 (&acc)[TM][TN]) {
  typedef typename Frag<T>::type frag_t;
  constexpr int KC = Frag<T>::KC, VEC = Frag<T>::VEC;
  frag_t fa[2][TM], fw[2][TN];
  const int k_lane = (lane >> 4) * VEC;
  auto load_half = [&](int h, int k) {
#pragma unroll
    for (int j = 0; j < TN; ++j) fw[h][j] = *reinterpret_cast<const frag_t*>(wrow[j] + k);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[h][i] = *reinterpret_cast<const frag_t*>(arow[i] + k);
  };
  auto load = [&](int t) {                         // this wavefront's t-th chunk
    const int k = (wave + t * NW) * 2 * KC + k_lane;
    load_half(0, k);
    load_half(1, k + KC);
  };
  auto product = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4 c = mma(mma(f32x4{0.f, 0.f, 0.f, 0.f}, fa[0][i], fw[0][j]), fa[1][i], fw[1][j]);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][v] += c[v];
      }
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int whole = K / (2 * KC), n = whole > wave ? (whole - wave + NW - 1) / NW : 0;
  if (n > 0) load(0);
  __builtin_amdgcn_sched_barrier(0);
  for (int t = 1; t < n; ++t) {
    product();
    load(t);
    __builtin_amdgcn_sched_barrier(0);             // (the loads stay behind the products: their registers are the same)
  }
  if (n > 0) product();
  if (whole * 2 * KC < K && whole % NW == wave) {  // the chunk that K cuts short: a lane's values are all inside K or all beyond it
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = (2 * whole + h) * KC + k_lane;
      load_half(h, min(k, K - VEC));
      if (k >= K) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fw[h][j] = frag_t{};
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[h][i] = frag_t{};
      }
    }
    product();
  }
}

// the wavefronts' stages; their sums take the same place afterwards
constexpr int red_bytes(int tn) { return NW * tn * RSTRIDE * (int)sizeof(float); }
constexpr int tile_lds(int tm, int tn) {
  return NW * stage_bytes(tm, tn) > red_bytes(tn) ? NW * stage_bytes(tm, tn) : red_bytes(tn);
}

// the eight wavefronts' sums of one element, stride floats apart, added as a tree (fewer roundings at full size)
__device__ __forceinline__ float wave_sums(const float* p, int stride) {
  const float a = (p[0] + p[stride]) + (p[2 * stride] + p[3 * stride]);
  const float b = (p[4 * stride] + p[5 * stride]) + (p[6 * stride] + p[7 * stride]);
  return a + b;
}
static_assert(NW == 8, "wave_sums adds eight");

// row n of the segments' weights laid one below the other, as n runs over the output columns
template <typename T, int EPI>
__device__ __forceinline__ const T* weight_row(const GemmArgs& a, int n) {
  n = min(n, a.N - 1);
  int s = 0;
  if (n >= a.Nseg[0] && EPI == EPI_STORE) {
    n -= a.Nseg[0];
    s = 1;
    if (n >= a.Nseg[1]) { n -= a.Nseg[1]; s = 2; }
  }
  return (const T*)(s == 0 ? a.W[0] : s == 1 ? a.W[1] : a.W[2]) + (size_t)n * a.K;
}

// output element (m, n) from its sums (SWIGLU: of gate and up)
template <typename T, int EPI>
__device__ __forceinline__ void store_element(const GemmArgs& a, bool has_bias, int m, int n, float s, float u) {
  if (EPI == EPI_SWIGLU) s = s / (1.f + __expf(-s)) * u;
  if (has_bias) {
    const bool s0 = n < a.Nseg[0], s1 = n < a.Nseg[0] + a.Nseg[1];
    const T* b = (const T*)(s0 ? a.bias[0] : s1 ? a.bias[1] : a.bias[2]);
    if (b) s += to_f32(b[s0 ? n : s1 ? n - a.Nseg[0] : n - a.Nseg[0] - a.Nseg[1]]);
  }
  if (EPI == EPI_RESID) s += to_f32(((const T*)a.R)[(size_t)m * a.ldc + n]);
  ((T*)a.C)[(size_t)m * a.ldc + n] = from_f32<T>(s);
}

// C tile of 16*TM rows x 16*TN columns (SWIGLU: TN/2 fragments of gate rows and the same rows of up)
template <typename T, int EPI, int TM, int TN, bool REGS>
__global__ __launch_bounds__(64 * NW) void tile_gemm_kernel(GemmArgs a) {
  extern __shared__ __align__(1024) unsigned char smem[];
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  float(*red)[TN][RSTRIDE] = reinterpret_cast<float(*)[TN][RSTRIDE]>(smem);
  constexpr int NO = EPI == EPI_SWIGLU ? TN / 2 : TN;      // output fragments along the columns
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int m_max = a.M_dev ? min(*a.M_dev, a.M) : a.M;
  const int m0 = blockIdx.y * 16 * TM, n0 = blockIdx.x * 16 * NO;
  if (m0 >= m_max) return;
  const int K = a.K;
  const auto tile_row = [&](int r) {               // row r of the tile's TM*16 activation and TN*16 weight rows
    if (r < 16 * TM) return (const T*)a.A + (size_t)min(m0 + r, m_max - 1) * a.lda;
    r -= 16 * TM;
    if (EPI == EPI_SWIGLU) return (const T*)(r < 16 * NO ? a.W[0] : a.W[1]) + (size_t)min(n0 + r % (16 * NO), a.N - 1) * K;
    return weight_row<T, EPI>(a, n0 + r);
  };
  f32x4 acc[TM][TN];
  if constexpr (REGS) {
    const T *arow[TM], *wrow[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) arow[i] = tile_row(16 * i + (lane & 15));
#pragma unroll
    for (int j = 0; j < TN; ++j) wrow[j] = tile_row(16 * (TM + j) + (lane & 15));
    tile_product_regs<T, TM, TN>(arow, wrow, K, wave, lane, acc);
  } else {
    const T* src[2 * (TM + TN)];
    tile_sources<T, TM, TN>(src, lane, tile_row);
    tile_product<T, TM, TN>(src, K, wave, lane, lds0 + wave * stage_bytes(TM, TN), acc);
  }
  const bool has_bias = EPI == EPI_STORE && (a.bias[0] || a.bias[1] || a.bias[2]);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    __syncthreads();                               // the sums go where the stages, or the last row's sums, were
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][j][v * 64 + lane] = acc[i][j][v];
    __syncthreads();
    for (int e = threadIdx.x; e < NO * 256; e += 64 * NW) {
      const int j = e >> 8, q = e & 255, el = q & 63;
      const int m = m0 + 16 * i + 4 * (el >> 4) + (q >> 6), n = n0 + 16 * j + (el & 15);
      if (m >= m_max || n >= a.N) continue;
      float s = wave_sums(&red[0][j][q], TN * RSTRIDE);
      // store_element, written out: called here it costs the smaller tiles with a bias 0.4 us a launch (128 x 1536, K = 1024)
      if (EPI == EPI_SWIGLU) {
        const float u = wave_sums(&red[0][j + NO][q], TN * RSTRIDE);
        s = s / (1.f + __expf(-s)) * u;
      }
      if (has_bias) {
        const bool s0 = n < a.Nseg[0], s1 = n < a.Nseg[0] + a.Nseg[1];
        const T* b = (const T*)(s0 ? a.bias[0] : s1 ? a.bias[1] : a.bias[2]);
        if (b) s += to_f32(b[s0 ? n : s1 ? n - a.Nseg[0] : n - a.Nseg[0] - a.Nseg[1]]);
      }
      if (EPI == EPI_RESID) s += to_f32(((const T*)a.R)[(size_t)m * a.ldc + n]);
      ((T*)a.C)[(size_t)m * a.ldc + n] = from_f32<T>(s);
    }
  }
}

// The same sums where K has at most six chunks: one wavefront per 32 x 32 output tile adds its chunks' products in the order
// of wave_sums (the other chunks' are zero), in registers.  With so few chunks some of the eight wavefronts of a shared tile
// have none, and the trip through LDS takes longer than the products.  MAX_CHUNKS: 4 (fewer registers), or 6 for five and six.
constexpr int SW = 4;      // wavefronts of a workgroup, side by side along the columns

template <typename T, int EPI, int MAX_CHUNKS>
__global__ __launch_bounds__(64 * SW) void tile_gemm_short_kernel(GemmArgs a, int col_blocks) {
  typedef typename Frag<T>::type frag_t;
  constexpr int KC = Frag<T>::KC, VEC = Frag<T>::VEC, TM = 2, NO = 2, TN = EPI == EPI_SWIGLU ? 2 * NO : NO;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l16 = lane & 15;
  const int m_max = a.M_dev ? min(*a.M_dev, a.M) : a.M;
  const int m0 = blockIdx.x / col_blocks * 16 * TM, n0 = (blockIdx.x % col_blocks * SW + wave) * 16 * NO;
  if (m0 >= m_max || n0 >= a.N) return;
  const int K = a.K;
  const T* arow[TM];
  const T* wrow[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) arow[i] = (const T*)a.A + (size_t)min(m0 + 16 * i + l16, m_max - 1) * a.lda;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    if (EPI == EPI_SWIGLU) wrow[j] = (const T*)a.W[j / NO] + (size_t)min(n0 + 16 * (j % NO) + l16, a.N - 1) * K;
    else wrow[j] = weight_row<T, EPI>(a, n0 + 16 * j + l16);
  }
  f32x4 sum[TM][TN], part[TM][TN];
  auto add_chunk = [&](int t, f32x4 (&to)[TM][TN]) {      // K is a multiple of 8: a lane's values are all inside K or beyond it
    frag_t fa[2][TM], fw[2][TN];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = (2 * t + h) * KC + (lane >> 4) * VEC, kk = min(k, K - VEC);
#pragma unroll
      for (int j = 0; j < TN; ++j) fw[h][j] = *reinterpret_cast<const frag_t*>(wrow[j] + kk);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[h][i] = *reinterpret_cast<const frag_t*>(arow[i] + kk);
      if (k >= K) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fw[h][j] = frag_t{};
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[h][i] = frag_t{};
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const f32x4 c = mma(mma(f32x4{0.f, 0.f, 0.f, 0.f}, fa[0][i], fw[0][j]), fa[1][i], fw[1][j]);
#pragma unroll
        for (int v = 0; v < 4; ++v) to[i][j][v] += c[v];
      }
  };
  auto clear = [&](f32x4 (&to)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) to[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto add = [&](f32x4 (&to)[TM][TN], const f32x4 (&x)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) to[i][j][v] += x[i][j][v];
  };
  const int chunks = (K + 2 * KC - 1) / (2 * KC);
  clear(sum);
  add_chunk(0, sum);
  if (chunks > 1) add_chunk(1, sum);
  if (chunks > 2) {
    clear(part);
    add_chunk(2, part);
    if (chunks > 3) add_chunk(3, part);
    add(sum, part);
  }
  if constexpr (MAX_CHUNKS > 4) {
    static_assert(MAX_CHUNKS <= 6, "the second half of the tree is (4 + 5) + 0");
    clear(part);
    add_chunk(4, part);
    if (chunks > 5) add_chunk(5, part);
    add(sum, part);
  }
  const bool has_bias = EPI == EPI_STORE && (a.bias[0] || a.bias[1] || a.bias[2]);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int j = 0; j < NO; ++j) {
        const int m = m0 + 16 * i + 4 * (lane >> 4) + v, n = n0 + 16 * j + l16;
        if (m < m_max && n < a.N) store_element<T, EPI>(a, has_bias, m, n, sum[i][j][v], EPI == EPI_SWIGLU ? sum[i][j + NO][v] : 0.f);
      }
}

// LM head: rows r < *count of n against vocabulary tiles of 64 tokens.  blockIdx.x = vocabulary part (tiles x, x + n_part,
// ..), blockIdx.y = group of 64 rows.  Every part leaves one (top, lowest index, runner-up, sum exp) summary per row.
template <typename T, int TM>
__device__ __forceinline__ void head_tiles(const T* n, const T* wv, int d, int V, float scale, int rows, int m0, int n_part,
                                           int m_cap, TopPartial* part, unsigned char* smem) {
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  float* red = reinterpret_cast<float*>(smem);
  constexpr int TN = 4, PER = TM * 16 / NW;        // tokens rows of the tile whose summaries one wavefront keeps
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15;
  float top_m[PER], top_m2[PER], top_s[PER];       // (an array of the structure ends up in scratch memory)
  int top_i[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const Top e = top_empty();
    top_m[p] = e.m; top_m2[p] = e.m2; top_s[p] = e.s; top_i[p] = e.idx;
  }
  const int tiles = (V + 16 * TN - 1) / (16 * TN);
  for (int t = blockIdx.x; t < tiles; t += n_part) {
    const T* src[2 * (TM + TN)];
    tile_sources<T, TM, TN>(src, lane, [&](int r) {
      return r < 16 * TM ? n + (size_t)min(m0 + r, rows - 1) * d : wv + (size_t)min(t * 16 * TN + r - 16 * TM, V - 1) * d;
    });
    f32x4 acc[TM][TN];
    if (t != (int)blockIdx.x) __syncthreads();     // the sums of the last tile lie where the stages are
    tile_product<T, TM, TN>(src, d, wave, lane, lds0 + wave * stage_bytes(TM, TN), acc);
    const int idx = t * 64 + lane;                 // this lane's token of the tile
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(wave * TN + j) * RSTRIDE + v * 64 + lane] = acc[i][j][v];
      __syncthreads();
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int m = wave * 2 + p;                // row within the fragment: element (m, token) of the tile
        const int q = (m & 3) * 64 + (m >> 2) * 16 + l16;
        float l = wave_sums(red + (lane >> 4) * RSTRIDE + q, TN * RSTRIDE);
        l = idx < V ? l * scale : -INFINITY;
        const float mx = wave_max(l);
        const unsigned long long at = __ballot(l == mx);
        const int win = at ? __ffsll((long long)at) - 1 : 0;
        Top one;
        one.m = mx;
        one.idx = t * 64 + win;
        one.m2 = wave_max(lane == win ? -INFINITY : l);
        one.s = wave_sum(l == -INFINITY ? 0.f : __expf(l - mx));
        const int c = i * 2 + p;
        one = top_merge(Top{top_m[c], top_m2[c], top_s[c], top_i[c]}, one);
        top_m[c] = one.m; top_m2[c] = one.m2; top_s[c] = one.s; top_i[c] = one.idx;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int r = m0 + 16 * i + wave * 2 + p;
      const int c = i * 2 + p;
      if (lane == 0 && r < rows) part[(size_t)blockIdx.x * m_cap + r] = TopPartial{top_m[c], top_m2[c], top_s[c], top_i[c]};
    }
}

// One workgroup to a CU (112 KB of LDS for 48 rows).  39 of 64 rows, fp32, 32000 x 1024: 45 us, 62 with fragments loaded into
// registers and the running summaries in scratch memory; the fp32 matrix pipes alone need 23 for the 48 rows computed.
template <typename T>
__global__ __launch_bounds__(64 * NW) void tile_head_kernel(const T* __restrict__ n, const T* __restrict__ wv, int d, int V,
                                                            float scale, const int32_t* __restrict__ count, int M, int m_cap,
                                                            TopPartial* __restrict__ part) {
  extern __shared__ __align__(1024) unsigned char smem[];
  const int rows = min(*count, M), m0 = blockIdx.y * 64;
  if (m0 >= rows) return;
  const int left = rows - m0, n_part = gridDim.x;
  // as many 16-row fragments as there are rows
  if (left > 48) head_tiles<T, 4>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, smem);
  else if (left > 32) head_tiles<T, 3>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, smem);
  else if (left > 16) head_tiles<T, 2>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, smem);
  else head_tiles<T, 1>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, smem);
}

template <typename T, int EPI, int TM, int TN, bool REGS = false>
hipError_t launch_tile(const GemmArgs& a, hipStream_t st) {
  constexpr int NO = EPI == EPI_SWIGLU ? TN / 2 : TN, LDS = REGS ? red_bytes(TN) : tile_lds(TM, TN);
  static std::atomic<unsigned long long> lds_ok{0};
  const hipError_t e = allow_dynamic_lds((const void*)tile_gemm_kernel<T, EPI, TM, TN, REGS>, LDS, lds_ok);
  if (e != hipSuccess) return e;
  tile_gemm_kernel<T, EPI, TM, TN, REGS><<<dim3(cdiv(a.N, 16 * NO), cdiv(a.M, 16 * TM)), 64 * NW, LDS, st>>>(a);
  return hipGetLastError();
}

template <typename T, int EPI, int MAX_CHUNKS>
void launch_short(const GemmArgs& a, hipStream_t st) {
  const int col_blocks = cdiv(a.N, 32 * SW);
  tile_gemm_short_kernel<T, EPI, MAX_CHUNKS><<<cdiv(a.M, 32) * col_blocks, 64 * SW, 0, st>>>(a, col_blocks);
}

// Tile shapes, measured, us:
// bf16 runs 64 x 64 tiles (SWIGLU: 32 features) where they fill the chip: a quarter of the operand traffic per product (4104
// columns, K = 1032: 200 rows, 260 tiles, 13.7, with 32 x 32 14.3, with 32 x 16 15.4; 1024 rows 44.7, 48.4, 56.9; 4096 rows 148, 175,
// 214).  fp32 has 64 x 64 tiles with fragments in registers, and 32 x 32 tiles in LDS, two workgroups a CU, one adding sums while
// the other multiplies.  The small ones win while K is short or the large ones leave a round of 256 workgroups half empty; with
// longer K the large ones' quarter of the traffic does (1024 columns of 2816, 1000 rows: 57 us, small 68; 11008 x 4104, 1000 rows
// 845, 1076, SwiGLU 3000 rows 5548, 7715; 1536 x 1024, 1000 rows 47, 39).  Of 1700 shapes measured (512 .. 11008 columns, K = 200 .. 8192,
// 256 .. 3500 large tiles) the line below is 0.3% over the better of both on average, large tiles alone 9%, small ones alone 5%.
// Below that 32 x 32 or 32 x 16 (SWIGLU: 16 features either way), by rounds of 256 workgroups: one of 32 x 32 takes as long as 1.6 of
// 32 x 16 in bf16, 1.9 in fp32, and starts sooner (K = 1024, 32 x 16 / 32 x 32: fp32 64 x 2048 6.3 / 8.6, 64 x 3072 9.8 / 8.9, 64 x 4104
// 13.4 / 15.4; bf16 64 x 1544 3.7 / 4.1, 128 x 1032 4.6 / 4.2, 128 x 2056 5.4 / 5.9).  16 x 16 with one fragment of rows.
// Where 64 x 64 tiles would fill the chip and K has up to six chunks in fp32 (192), four in bf16 (256), a wavefront takes a
// tile: 4096 x 4104 from K = 8 78 -> 23 / 67 -> 14, K = 136 112 -> 82 / 70 -> 32; with more chunks the shared tiles were as fast
// or faster where they just fill the chip (1024 x 1032, SwiGLU: seven chunks fp32 23 against 25, five bf16 15 against 18).
template <typename T, int EPI>
hipError_t launch_epi(const GemmArgs& a, hipStream_t st) {
  constexpr int CHUNK = 2 * Frag<T>::KC;
  constexpr bool F32 = sizeof(T) == 4;
  const int big = cdiv(a.M, 64) * cdiv(a.N, EPI == EPI_SWIGLU ? 32 : 64);
  if (big >= 256 && a.K <= 4 * CHUNK) {
    launch_short<T, EPI, 4>(a, st);
    return hipGetLastError();
  }
  if (F32 && big >= 256 && a.K <= 6 * CHUNK) {
    launch_short<float, EPI, 6>(a, st);
    return hipGetLastError();
  }
  if constexpr (!F32)
    if (big >= 256) return launch_tile<T, EPI, 4, 4>(a, st);
  const int rows = cdiv(a.M, 32), r16 = cdiv(rows * cdiv(a.N, 16), 256), r32 = cdiv(rows * cdiv(a.N, 32), 256);
  if constexpr (F32) {
    const float large = 0.7f * cdiv(big, 256) + 0.3f * (big / 256.f), small = EPI == EPI_SWIGLU ? r16 : r32;    // rounds of either tile
    if (big >= 256 && 3.05f * large * (a.K + 800.f) <= small * (a.K + 400.f)) return launch_tile<T, EPI, 4, 4, true>(a, st);
  }
  if (a.M <= 16) return launch_tile<T, EPI, 1, EPI == EPI_SWIGLU ? 2 : 1>(a, st);
  if (EPI == EPI_SWIGLU || (F32 ? 19 * r32 - 2 < 10 * r16 : 16 * r32 < 10 * r16)) return launch_tile<T, EPI, 2, 2>(a, st);
  if constexpr (EPI != EPI_SWIGLU) return launch_tile<T, EPI, 2, 1>(a, st);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_t(int epi, const GemmArgs& a, hipStream_t st) {
  switch (epi) {
    case EPI_STORE: return launch_epi<T, EPI_STORE>(a, st);
    case EPI_RESID: return launch_epi<T, EPI_RESID>(a, st);
    case EPI_SWIGLU: return launch_epi<T, EPI_SWIGLU>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_gemm_tile(int dtype, int epi, const GemmArgs& a, hipStream_t st) {
  return dtype == SPIFFY_F32 ? launch_t<float>(epi, a, st) : launch_t<bf16_t>(epi, a, st);
}

hipError_t launch_lmhead_tile(int dtype, const void* n, const void* w_vocab, int d, int V, float scale, const int32_t* count,
                              int M, int m_cap, int n_part, TopPartial* part, hipStream_t st) {
  const dim3 grid(n_part, cdiv(M, 64));
  const int lds = tile_lds(M > 48 ? 4 : cdiv(M, 16), 4);      // for as many 16-row fragments as there can be
  static std::atomic<unsigned long long> lds_ok[2];
  hipError_t e;
  if (dtype == SPIFFY_F32) {
    if ((e = allow_dynamic_lds((const void*)tile_head_kernel<float>, tile_lds(4, 4), lds_ok[0])) != hipSuccess) return e;
    tile_head_kernel<float><<<grid, 64 * NW, lds, st>>>((const float*)n, (const float*)w_vocab, d, V, scale, count, M, m_cap, part);
  } else {
    if ((e = allow_dynamic_lds((const void*)tile_head_kernel<bf16_t>, tile_lds(4, 4), lds_ok[1])) != hipSuccess) return e;
    tile_head_kernel<bf16_t><<<grid, 64 * NW, lds, st>>>((const bf16_t*)n, (const bf16_t*)w_vocab, d, V, scale, count, M, m_cap,
                                                          part);
  }
  return hipGetLastError();
}

}  // namespace spiffy
