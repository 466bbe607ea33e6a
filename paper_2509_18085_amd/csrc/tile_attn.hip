// Block attention for every shape and type the head_dim-128 bf16 kernel does not take: any head_dim that is a multiple of 8
// up to 256, fp32 or bf16 storage.  Scores, probabilities and sums are fp32 throughout (v_mfma_f32_16x16x4_f32): rotated
// queries and own keys are never rounded to bf16 here.
//
// keys of a query of state g = [P cached keys ; the B keys of state g ; S cached keys of the tokens after the block (dual
// cache)], bidirectional inside the block (Fig. 4); cache row j holds sequence position j, so rows P .. P+B-1 of the cache
// (the slot of the block itself) are never read.
//
// The work is small (a few hundred keys) and bound by latency.  One workgroup = 16 query rows of one (state, KV head): the
// query heads of a group share their K and V rows.  Its eight wavefronts take 16-key chunks in turn (chunk c to wavefront
// c % 8), each with a running maximum of its own, and merge through LDS in wavefront order.  A wavefront computes
// S^T = K Q^T and then O^T = V^T P^T: accumulator element v of lane (q = lane % 16, group = lane / 16) of S^T is key
// 4 * group + v of query q, which is exactly the P^T operand element of the second product's v-th step, so the
// probabilities never leave their registers, and the softmax scale of a query is lane-local in both products.
// Values are loaded in front of the scores and kept as they are stored, so that they arrive meanwhile.  Loading keys and values a
// whole chunk ahead was measured and taken back: bf16, 128 workgroups, 17.7 us with it and 17.3 without at 544 keys of 64, 13.6 and
// 12.5 at 232, 31.4 and 30.6 at 544 keys of 128.  Above head_dim 128 in fp32 a wavefront spills 18 to 118 registers (bf16 above 192:
// 34), shapes that only have to run.
// Measured against one workgroup per (row, head), which computed its own rotary angles in double precision and read K one
// row per thread: bf16, 128 rows, 16 heads of 64, 544 keys 102 -> 17.3 us; what is left is the fp32 matrix rate on 128
// workgroups and the latency of a chunk.
#include "kernels.h"

namespace spiffy {

namespace {

constexpr int NW = 8;

// four values as they are stored, and as fp32
template <typename T> struct Four;
template <> struct Four<float> { typedef f32x4 type; };
template <> struct Four<bf16_t> { typedef bf16x4 type; };
template <typename T> __device__ __forceinline__ typename Four<T>::type load4_raw(const T* p) {
  return *reinterpret_cast<const typename Four<T>::type*>(p);
}
__device__ __forceinline__ f32x4 widen(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 widen(bf16x4 v) {
  return f32x4{static_cast<float>(v[0]), static_cast<float>(v[1]), static_cast<float>(v[2]), static_cast<float>(v[3])};
}
template <typename T> __device__ __forceinline__ f32x4 load4(const T* p) { return widen(load4_raw(p)); }

// values k .. k+3 of a row rotated by the angles of table row `tab` [half] (k % 4 == 0, half % 4 == 0)
template <typename T>
__device__ __forceinline__ f32x4 load4_rotated(const T* row, int k, int half, const float2* tab) {
  const bool low = k < half;
  const int f = low ? k : k - half;
  const f32x4 x = load4(row + k), y = load4(row + (low ? k + half : k - half));
  const f32x4 t0 = *reinterpret_cast<const f32x4*>(tab + f), t1 = *reinterpret_cast<const f32x4*>(tab + f + 2);
  const float c[4] = {t0[0], t0[2], t1[0], t1[2]}, s[4] = {t0[1], t0[3], t1[1], t1[3]};
  f32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = low ? x[e] * c[e] - y[e] * s[e] : x[e] * c[e] + y[e] * s[e];
  return r;
}

// H64 = head_dim in units of 64, rounded up; rows of Q, K, V beyond head_dim count as zero
template <typename T, int H64>
__global__ __launch_bounds__(64 * NW) void tile_attn_kernel(const T* __restrict__ qkv, const T* __restrict__ pk,
                                                            const T* __restrict__ pv, T* __restrict__ out,
                                                            const float2* __restrict__ tab, int B, int Hq, int Hkv, int hd,
                                                            int P, int S, int ldp, int own) {
  constexpr int NQ = 4 * H64;                       // 16-wide K steps of Q K^T
  extern __shared__ float smem[];                   // merge buffer [NW][16][hd + 2]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, grp = lane >> 4;
  const int half = hd >> 1, rep = Hq / Hkv, ld = (Hq + 2 * Hkv) * hd;
  const int tiles = (B * rep + 15) / 16;
  const int qt = blockIdx.x % tiles, kvh = (blockIdx.x / tiles) % Hkv, g = blockIdx.x / (tiles * Hkv);
  const int row = min(qt * 16 + l16, B * rep - 1);  // (position, head of the group) of this lane's query
  const int b = row / rep, h = kvh * rep + row % rep;
  const T* qrow = qkv + (size_t)(g * B + b) * ld + h * hd;
  const float scale = 1.0f / sqrtf((float)hd);
  const int n_keys = own ? P + B + S : P;           // own == 0: cache rows 0 .. P-1 only
  const int chunks = (n_keys + 15) / 16;
  float m = -INFINITY, sum = 0.f;
  f32x4 o[H64][4];                                  // O^T: rows 64 * u + 4 * (row of the fragment) + j, column q
#pragma unroll
  for (int u = 0; u < H64; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) o[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // A chunk's keys (lane: key l16, values 16 * i + 4 * grp ..) and values (lane: keys 4 * grp + v, dims 64 * u + 4 * l16 ..)
  typedef typename Four<T>::type four_t;
  struct Chunk {
    four_t k[NQ], v[4][H64];
  };
  auto touches_block = [&](int c) { return 16 * c < P + B && 16 * c + 16 > P && n_keys > P; };
  auto load_values = [&](int c, Chunk& ch) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 16 * c + 4 * grp + v;
      const bool in_block = j >= P && j < P + B;
      const T* vr = in_block ? qkv + (size_t)(g * B + (j - P)) * ld + (Hq + Hkv + kvh) * hd : pv + ((size_t)kvh * ldp + j) * hd;
#pragma unroll
      for (int u = 0; u < H64; ++u) {
        const int t = 64 * u + 4 * l16;
        ch.v[v][u] = j < n_keys && t < hd ? load4_raw(vr + t) : four_t{};
      }
    }
  };
  auto load_keys = [&](int c, Chunk& ch) {          // cached keys; own keys are rotated and read where they are used
    const T* kr = pk + ((size_t)kvh * ldp + min(16 * c + l16, n_keys - 1)) * hd;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int k = 16 * i + 4 * grp;
      ch.k[i] = k < hd ? load4_raw(kr + k) : four_t{};
    }
  };
  Chunk cur;
  f32x4 q[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int k = 16 * i + 4 * grp;
    q[i] = k < hd ? load4_rotated(qrow, k, half, tab + (size_t)b * half) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int c = wave; c < chunks; c += NW) {
    load_values(c, cur);                            // in flight during the scores
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (touches_block(c)) {
      const int jk = min(16 * c + l16, n_keys - 1);   // this lane's key (operand rows beyond the last key repeat it)
      const bool in_block = jk >= P && jk < P + B;
      const int bb = in_block ? jk - P : 0;
      const T* kr = in_block ? qkv + (size_t)(g * B + bb) * ld + (Hq + kvh) * hd : pk + ((size_t)kvh * ldp + jk) * hd;
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int k = 16 * i + 4 * grp;
        f32x4 kk = {0.f, 0.f, 0.f, 0.f};
        if (k < hd) {
          if (in_block) kk = load4_rotated(kr, k, half, tab + (size_t)bb * half);
          else kk = load4(kr + k);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kk[e], q[i][e], s, 0, 0, 0);
      }
    } else {
      load_keys(c, cur);
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const f32x4 kk = widen(cur.k[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kk[e], q[i][e], s, 0, 0, 0);
      }
    }
    float mc = m;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      s[v] = 16 * c + 4 * grp + v < n_keys ? s[v] * scale : -INFINITY;
      mc = fmaxf(mc, s[v]);
    }
    const auto larger = [](float x, float y) { return fmaxf(x, y); };
    mc = reduce_32(reduce_16(mc, larger), larger);
    const float f = m == -INFINITY ? 0.f : __expf(m - mc);     // nothing accumulated yet: the sums are zero
    float ps = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      s[v] = s[v] == -INFINITY ? 0.f : __expf(s[v] - mc);
      ps += s[v];
    }
    m = mc;
    sum = sum * f + ps;                             // this lane's keys only; the four groups meet at the end
#pragma unroll
    for (int u = 0; u < H64; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[u][j][e] *= f;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          o[u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(static_cast<float>(cur.v[v][u][j]), s[v], o[u][j], 0, 0, 0);
      }
  }
  const auto plus = [](float x, float y) { return x + y; };
  sum = reduce_32(reduce_16(sum, plus), plus);
  // merge through LDS: every wavefront leaves its sums, then all threads add the eight of an output element in order
  const int ldm = hd + 2;
  {
    float* dst = smem + (wave * 16 + l16) * ldm;
#pragma unroll
    for (int u = 0; u < H64; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int t = 64 * u + 4 * (4 * grp + v) + j;
          if (t < hd) dst[t] = o[u][j][v];
        }
    if (grp == 0) { dst[hd] = m; dst[hd + 1] = sum; }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * hd; e += 64 * NW) {
    const int qi = e / hd, t = e % hd;
    const int r = qt * 16 + qi;
    if (r >= B * rep) break;
    const float* src = smem + qi * ldm;
    float mm = src[hd];
#pragma unroll
    for (int w = 1; w < NW; ++w) mm = fmaxf(mm, src[w * 16 * ldm + hd]);
    float val = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* sw = src + w * 16 * ldm;
      const float f = sw[hd] == -INFINITY ? 0.f : __expf(sw[hd] - mm);    // a wavefront without keys
      val += sw[t] * f;
      den += sw[hd + 1] * f;
    }
    out[(size_t)(g * B + r / rep) * (Hq * hd) + (kvh * rep + r % rep) * hd + t] = from_f32<T>(val / den);
  }
}

template <typename T, int H64>
hipError_t launch_h(const AttnArgs& a, hipStream_t st) {
  const int grid = a.G * a.Hkv * cdiv(a.B * (a.Hq / a.Hkv), 16);
  const size_t smem = sizeof(float) * NW * 16 * (size_t)(a.hd + 2);
  if (smem > 64 * 1024) {
    static std::atomic<unsigned long long> lds_ok{0};
    const hipError_t e = allow_dynamic_lds((const void*)tile_attn_kernel<T, H64>,
                                           (int)(sizeof(float) * NW * 16 * (64 * H64 + 2)), lds_ok);
    if (e != hipSuccess) return e;
  }
  tile_attn_kernel<T, H64><<<grid, 64 * NW, smem, st>>>((const T*)a.qkv, (const T*)a.prefix_k, (const T*)a.prefix_v,
                                                        (T*)a.out, (const float2*)a.partial, a.B, a.Hq, a.Hkv, a.hd,
                                                        a.P, a.S, a.ldp ? a.ldp : a.P, a.own);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const AttnArgs& a, hipStream_t st) {
  switch (cdiv(a.hd, 64)) {
    case 1: return launch_h<T, 1>(a, st);
    case 2: return launch_h<T, 2>(a, st);
    case 3: return launch_h<T, 3>(a, st);
    default: return launch_h<T, 4>(a, st);
  }
}

}  // namespace

hipError_t launch_attn_tile(int dtype, const AttnArgs& a, hipStream_t st) {
  return dtype == SPIFFY_F32 ? launch_t<float>(a, st) : launch_t<bf16_t>(a, st);
}

}  // namespace spiffy
