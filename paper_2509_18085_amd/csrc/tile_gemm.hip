// GEMM and LM head for every shape and type the bf16 MFMA GEMM does not take: fp32 operands, bf16 widths that do not fill
// its 64-wide K tiles.  fp32 operands run on v_mfma_f32_16x16x4_f32 (fp32 products, fp32 sums: the arithmetic of a chain of
// fused multiply-adds), bf16 operands on v_mfma_f32_16x16x32_bf16.
//
// What bounds these shapes: with the 16 - 128 rows of a few states, the requests for weight and activation lines that a CU
// keeps in flight, and the latency of the chain of loads along K; with several hundred rows the fp32 matrix pipes (256
// flop per clock and CU).  Both operands are K-contiguous, and a 16x16 fragment of either type is one 16-byte load per lane
// whose four lane groups read 64 contiguous bytes of a row, so nothing is staged in LDS: every wavefront loads fragments
// straight into a ring of DEPTH register buffers.  Eight wavefronts share one output tile and split K (chunk c of 128
// bytes, a whole line of each row, goes to wavefront c % 8), which puts eight times as many loads in flight per tile;
// their sums are added through LDS as a fixed tree.  The K order of an element depends on K alone, not on the tile or
// on M, so a row's result does not depend on the rows computed with it.
//
// Measured, against a 64x64-tile kernel on vector FMAs with scalar loads (and, for the head, one workgroup per row that
// streamed the whole vocabulary matrix): bf16, 128 rows, width 1024, FFN 2816: QKV 334 -> 9.8 us (three launches -> one),
// gate/up 208 -> 14.6, output and down 8.2 on average.  fp32, 39 of 64 rows against 32000 tokens x 1024: 44 ms -> 62 us.
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

// One output tile: rows m0 .. m0+16*TM-1 (below m_max), weight rows given by `wrow` (TN fragments of 16).
// On return wavefront 0's .. 7's sums are in acc; the caller reduces them.
template <typename T, int TM, int TN, int DEPTH>
__device__ __forceinline__ void tile_product(const T* const (&arow)[TM], const T* const (&wrow)[TN], int K, int wave, int lane,
                                             f32x4 (&acc)[TM][TN]) {
  typedef typename Frag<T>::type frag_t;
  constexpr int KC = Frag<T>::KC, VEC = Frag<T>::VEC;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  frag_t fa[DEPTH][2][TM], fw[DEPTH][2][TN];
  const int k_lane = (lane >> 4) * VEC;
  auto load_half = [&](int buf, int h, int k) {
#pragma unroll
    for (int j = 0; j < TN; ++j) fw[buf][h][j] = *reinterpret_cast<const frag_t*>(wrow[j] + k);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[buf][h][i] = *reinterpret_cast<const frag_t*>(arow[i] + k);
  };
  auto load = [&](int buf, int t) {                // this wavefront's t-th chunk
    const int k = (wave + t * NW) * 2 * KC + k_lane;
    load_half(buf, 0, k);
    load_half(buf, 1, k + KC);
  };
  // fp32: a chunk's products are summed on their own and then added, so that the long sum along K is rounded once a chunk
  // and wavefront (a layer of width 1024 against 64 bits: 5.0e-7 with one chain, 3.0e-7 so; no measurable time)
  auto product = [&](int buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (std::is_same<T, float>::value) {
          f32x4 c = mma(f32x4{0.f, 0.f, 0.f, 0.f}, fa[buf][0][i], fw[buf][0][j]);
          c = mma(c, fa[buf][1][i], fw[buf][1][j]);
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] += c[v];
        } else {
          acc[i][j] = mma(acc[i][j], fa[buf][0][i], fw[buf][0][j]);
          acc[i][j] = mma(acc[i][j], fa[buf][1][i], fw[buf][1][j]);
        }
      }
  };
  // whole chunks of this wavefront; every branch is wavefront-uniform
  const int whole = K / (2 * KC), n = whole > wave ? (whole - wave + NW - 1) / NW : 0;
#pragma unroll
  for (int s = 0; s < DEPTH; ++s)
    if (s < n) load(s, s);
  __builtin_amdgcn_sched_barrier(0);
  int t = 0;
  for (; t + 2 * DEPTH <= n; t += DEPTH) {
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      product(s);
      load(s, t + s + DEPTH);
      __builtin_amdgcn_sched_barrier(0);           // keep the ring: left alone, the scheduler gathers all loads at the end
    }
  }
#pragma unroll
  for (int s = 0; s < DEPTH; ++s) {
    if (t + s < n) product(s);
    if (t + s + DEPTH < n) load(s, t + s + DEPTH);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int s = 0; s < DEPTH - 1; ++s)
    if (t + s + DEPTH < n) product(s);
  // a last chunk that K cuts short: K is a multiple of 8, so a lane's values are all inside K or all beyond it
  if (whole * 2 * KC < K && whole % NW == wave) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = (2 * whole + h) * KC + k_lane;
      load_half(0, h, min(k, K - VEC));
      if (k >= K) {
#pragma unroll
        for (int j = 0; j < TN; ++j) fw[0][h][j] = frag_t{};
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[0][h][i] = frag_t{};
      }
    }
    product(0);
  }
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
template <typename T, int EPI, int TM, int TN, int DEPTH>
__global__ __launch_bounds__(64 * NW) void tile_gemm_kernel(GemmArgs a) {
  __shared__ float red[NW][TN][RSTRIDE];
  constexpr int NO = EPI == EPI_SWIGLU ? TN / 2 : TN;      // output fragments along the columns
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l16 = lane & 15;
  const int m_max = a.M_dev ? min(*a.M_dev, a.M) : a.M;
  const int m0 = blockIdx.y * 16 * TM, n0 = blockIdx.x * 16 * NO;
  if (m0 >= m_max) return;
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
  f32x4 acc[TM][TN];
  tile_product<T, TM, TN, DEPTH>(arow, wrow, K, wave, lane, acc);

  const bool has_bias = EPI == EPI_STORE && (a.bias[0] || a.bias[1] || a.bias[2]);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (i) __syncthreads();
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
                                           int m_cap, TopPartial* part, float* red) {
  constexpr int TN = 4, PER = TM * 16 / NW;        // tokens rows of the tile whose summaries one wavefront keeps
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15;
  const T* arow[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) arow[i] = n + (size_t)min(m0 + 16 * i + l16, rows - 1) * d;
  Top top[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) top[p] = top_empty();
  const int tiles = (V + 16 * TN - 1) / (16 * TN);
  for (int t = blockIdx.x; t < tiles; t += n_part) {
    const T* wrow[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) wrow[j] = wv + (size_t)min(t * 16 * TN + 16 * j + l16, V - 1) * d;
    f32x4 acc[TM][TN];
    tile_product<T, TM, TN, 1>(arow, wrow, d, wave, lane, acc);
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
        top[i * 2 + p] = top_merge(top[i * 2 + p], one);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int r = m0 + 16 * i + wave * 2 + p;
      const Top& o = top[i * 2 + p];
      if (lane == 0 && r < rows) part[(size_t)blockIdx.x * m_cap + r] = TopPartial{o.m, o.m2, o.s, o.idx};
    }
}

// One workgroup to a CU: 256 registers in fp32, 196 in bf16, for four row fragments, and the compiler keeps 160 bytes a lane in
// scratch memory.  Measured, 39 of 64 rows, fp32, 32000 x 1024: 62 us, 2.1 TB/s, bound by 64-byte segments of weight rows in
// flight from one workgroup.
template <typename T>
__global__ __launch_bounds__(64 * NW) void tile_head_kernel(const T* __restrict__ n, const T* __restrict__ wv, int d, int V,
                                                            float scale, const int32_t* __restrict__ count, int M, int m_cap,
                                                            TopPartial* __restrict__ part) {
  __shared__ float red[NW * 4 * RSTRIDE];
  const int rows = min(*count, M), m0 = blockIdx.y * 64;
  if (m0 >= rows) return;
  const int left = rows - m0, n_part = gridDim.x;
  // as many 16-row fragments as there are rows
  if (left > 48) head_tiles<T, 4>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, red);
  else if (left > 32) head_tiles<T, 3>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, red);
  else if (left > 16) head_tiles<T, 2>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, red);
  else head_tiles<T, 1>(n, wv, d, V, scale, rows, m0, n_part, m_cap, part, red);
}

template <typename T, int EPI, int MAX_CHUNKS>
void launch_short(const GemmArgs& a, hipStream_t st) {
  const int col_blocks = cdiv(a.N, 32 * SW);
  tile_gemm_short_kernel<T, EPI, MAX_CHUNKS><<<cdiv(a.M, 32) * col_blocks, 64 * SW, 0, st>>>(a, col_blocks);
}

// Tiles of 64 x 64 (SWIGLU: 32 features) where they fill the chip: a quarter of the operand traffic per product.  Below
// that 32 x 16 (16 x 16 with one fragment of rows): four to eight times the workgroups, each reading its operands once.
// Measured around the line, fp32 / bf16, in us with 64 x 64 and with 32 x 16: 200 rows of 4104 columns (260 tiles of 64 x 64),
// K = 1032: 45.4, 37.4 / 13.5, 17.9, SwiGLU 66, 58 / 22, 25; 1024 rows of 4104, 1040 tiles: 116, 150 / 46, 72; 4096 rows: 393,
// 578 / 148, 271 (one line for both types: fp32 alone would gain from 32 x 16 tiles a little longer).
// Where 64 x 64 tiles fill the chip and K has up to six chunks in fp32 (192), four in bf16 (256), a wavefront takes a tile: 4096 x
// 4104 from K = 8 87 -> 23 / 59 -> 15, K = 136 127 -> 81 / 65 -> 32; with more chunks the shared tiles were as fast or faster
// where they just fill the chip (1024 x 1032, SwiGLU: seven chunks fp32 23 against 25, five bf16 15 against 18).
template <typename T, int EPI>
hipError_t launch_epi(const GemmArgs& a, hipStream_t st) {
  constexpr int CHUNK = 2 * Frag<T>::KC;
  const int big = cdiv(a.M, 64) * cdiv(a.N, EPI == EPI_SWIGLU ? 32 : 64);
  if (big >= 256 && a.K <= 4 * CHUNK) {
    launch_short<T, EPI, 4>(a, st);
  } else if (big >= 256 && a.K <= 6 * CHUNK && sizeof(T) == 4) {
    launch_short<float, EPI, 6>(a, st);
  } else if (big >= 256) {
    constexpr int NO = EPI == EPI_SWIGLU ? 2 : 4;
    tile_gemm_kernel<T, EPI, 4, 4, 1><<<dim3(cdiv(a.N, 16 * NO), cdiv(a.M, 64)), 64 * NW, 0, st>>>(a);
  } else if (a.M <= 16) {
    tile_gemm_kernel<T, EPI, 1, EPI == EPI_SWIGLU ? 2 : 1, 2><<<dim3(cdiv(a.N, 16), 1), 64 * NW, 0, st>>>(a);
  } else {
    tile_gemm_kernel<T, EPI, 2, EPI == EPI_SWIGLU ? 2 : 1, 2><<<dim3(cdiv(a.N, 16), cdiv(a.M, 32)), 64 * NW, 0, st>>>(a);
  }
  return hipGetLastError();
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
  if (dtype == SPIFFY_F32)
    tile_head_kernel<float><<<grid, 64 * NW, 0, st>>>((const float*)n, (const float*)w_vocab, d, V, scale, count, M, m_cap, part);
  else
    tile_head_kernel<bf16_t><<<grid, 64 * NW, 0, st>>>((const bf16_t*)n, (const bf16_t*)w_vocab, d, V, scale, count, M, m_cap,
                                                       part);
  return hipGetLastError();
}

}  // namespace spiffy
