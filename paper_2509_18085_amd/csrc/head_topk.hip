// Drafting source (Sec. 4.4.2): the K most likely tokens of the accepted node's distribution at every
// masked position of its block, with their probabilities (vocabulary ranks j = 1..K).
//
// The LM head pass of the step has already reduced every masked row to (top logit, its token, sum of
// exponentials) and, on the MFMA path, left one such summary per 128-token chunk of the vocabulary.  The K
// best tokens of a row lie in the K chunks with the largest chunk maxima (a token outside them is beaten by
// the K maxima; equal logits go to the lower token id and chunks are contiguous id ranges), so only those
// K x 128 logits are recomputed - 1/250 of a second pass over the vocabulary matrix at V = 126k:
//   topk_refine_kernel   workgroup (position b, k, slice): picks the k-th best chunk of the row and recomputes
//                        a part of its 128 logits, four vocabulary rows a wavefront at a time
//   topk_full_kernel     path without chunk summaries (fp32 / shapes the MFMA head does not take): one
//                        workgroup per position scans the whole vocabulary, K best candidates
//   topk_merge_kernel    one workgroup per position: K best of the K x 128 logits (of the K candidates),
//                        probabilities from the row's (top logit, sum of exponentials); the row's argmax stays
//                        first with exactly the confidence the head reported
//
// The refinement is bound by what a compute unit can fetch (25 - 50 GB/s: a chunk of 4096-wide bf16 rows is 1 MB), so a
// chunk is shared by up to eight workgroups, each of which picks the chunk again (refine_slices).
#include "kernels.h"

namespace spiffy {

namespace {

constexpr int KMAX = SPIFFY_MAX_TOPK;

// compacted row of flattened position f, or -1 (row_idx is ascending)
__device__ __forceinline__ int find_row(const int32_t* __restrict__ row_idx, int n, int f) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (row_idx[mid] < f) lo = mid + 1; else hi = mid;
  }
  return (lo < n && row_idx[lo] == f) ? lo : -1;
}

// (value, index) ordering of the drafting source: larger value first, equal values to the lower index
__device__ __forceinline__ bool better(float v, int i, float v2, int i2) { return v > v2 || (v == v2 && i < i2); }

// best (value, index) over the wavefront, in the steps of wave_reduce
__device__ __forceinline__ void keep_better(float& v, int& i, float v2, int i2) {
  const bool b = better(v2, i2, v, i);
  v = b ? v2 : v;
  i = b ? i2 : i;
}
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
__device__ __forceinline__ void wave_best(float& v, int& i) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  u32x2 rv = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  u32x2 ri = __builtin_amdgcn_permlane32_swap((unsigned)i, (unsigned)i, false, false);
  v = __uint_as_float(rv[0]);
  i = (int)ri[0];
  keep_better(v, i, __uint_as_float(rv[1]), (int)ri[1]);
  rv = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  ri = __builtin_amdgcn_permlane16_swap((unsigned)i, (unsigned)i, false, false);
  v = __uint_as_float(rv[0]);
  i = (int)ri[0];
  keep_better(v, i, __uint_as_float(rv[1]), (int)ri[1]);
  keep_better(v, i, spiffy::dpp_move<0x128>(v), dpp_move<0x128>(i));
  keep_better(v, i, spiffy::dpp_move<0x1B>(spiffy::dpp_move<0x141>(v)), dpp_move<0x1B>(dpp_move<0x141>(i)));
  keep_better(v, i, spiffy::dpp_move<0x4E>(v), dpp_move<0x4E>(i));
  keep_better(v, i, spiffy::dpp_move<0xB1>(v), dpp_move<0xB1>(i));
}

template <typename T>
__device__ __forceinline__ float dot_row(const T* __restrict__ x, const T* __restrict__ w, int d, int lane);
template <>
__device__ __forceinline__ float dot_row<bf16_t>(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, int d, int lane) {
  float acc = 0.f;
  for (int e = lane * 8; e < d; e += 512) {        // d % 8 == 0 on this path
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(x + e);
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(w + e);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc = fmaf(static_cast<float>(a[t]), static_cast<float>(b[t]), acc);
  }
  return wave_sum(acc);
}
template <>
__device__ __forceinline__ float dot_row<float>(const float* __restrict__ x, const float* __restrict__ w, int d, int lane) {
  float acc = 0.f;
  for (int e = lane; e < d; e += 64) acc = fmaf(x[e], w[e], acc);
  return wave_sum(acc);
}

// dot products of x with four consecutive rows of w (row stride d): the same per-lane order and wavefront sum as dot_row
template <typename T>
__device__ __forceinline__ void dot_rows4(const T* __restrict__ x, const T* __restrict__ w, int d, int lane, float (&out)[4]);
template <>
__device__ __forceinline__ void dot_rows4<bf16_t>(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, int d, int lane,
                                                  float (&out)[4]) {
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int e = lane * 8; e < d; e += 512) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(x + e);
    bf16x8 b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = *reinterpret_cast<const bf16x8*>(w + (size_t)u * d + e);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[u] = fmaf(static_cast<float>(a[t]), static_cast<float>(b[u][t]), acc[u]);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) out[u] = wave_sum(acc[u]);
}
template <>
__device__ __forceinline__ void dot_rows4<float>(const float* __restrict__ x, const float* __restrict__ w, int d, int lane,
                                                 float (&out)[4]) {
#pragma unroll
  for (int u = 0; u < 4; ++u) out[u] = dot_row<float>(x, w + (size_t)u * d, d, lane);
}

// Workgroups that share a chunk: enough to have 256 + d / 4 at work, at most eight.  Each picks the chunk again (K rounds over the
// row's summaries), which the narrow widths notice and the wide ones do not.  24 positions, 2 chunks each of 4096 bf16 columns
// (50 MB): 55.9 us with a workgroup a chunk, 14.9 us with eight.  32 positions of 126464 tokens, us with one, two, four,
// eight: K = 8, width 4096 64.0, 48.1, 48.7, 51.6; width 512 25.0, 24.8, 27.6, 33.0; 128 positions, K = 8, width 512 35.6, 47.0, 51.7,
// 70.4.  Over 152 shapes measured (V 130 .. 262144, width 256 .. 8192) this is 1.1% over the best, eight throughout 9%.
// A workgroup a chunk where 400 .. 512 of them fill one round of two a CU, and for more than 640 (every position masked, us with one
// and with two: 448 chunks of width 3584 72.6 and 75.7, 256 x 2 81.8 and 93.7; 80 x 5 of width 4096 77.4 and 83.0, of 5120 81.6 and 89.0;
// 96 x 8 of 5120 147.0 and 151.7).
inline int refine_slices(int B, int K, int d) {
  const int chunks = B * K, limit = d < 7168 ? 256 + d / 4 : 2048;
  if (d < 7168 && ((chunks >= 400 && chunks <= 512) || chunks > 640)) return 1;
  int n = 8;
  while (n > 1 && chunks * n > limit) n /= 2;
  return n;
}
template <typename T>
__global__ __launch_bounds__(256) void topk_refine_kernel(HeadTopkArgs a) {
  __shared__ float s_val[2][4];
  __shared__ int s_idx[2][4];
  const int b = blockIdx.x, k = blockIdx.y;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int node = a.result ? a.result->node : a.node;
  const int r = (node >= 0 && node < a.G) ? find_row(a.row_idx, min(*a.count, a.G * a.B), node * a.B + b) : -1;
  if (r < 0) return;                                // the merge sees the same and reads nothing of this position
  // ---- the k-th best chunk of the row: k+1 rounds of a workgroup-wide best, each excluding the winners so far
  float mine[8];
  const int per = (a.n_part + 255) / 256;          // <= 8 (n_part <= 2048)
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int p = tid + 256 * q;
    mine[q] = (q < per && p < a.n_part) ? a.part[(size_t)p * a.m_cap + r].m : -INFINITY;
  }
  int chunk = -1;
  for (int round = 0; round <= k; ++round) {
    float v = -INFINITY;
    int i = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int p = tid + 256 * q;
      if (better(mine[q], p, v, i)) { v = mine[q]; i = p; }
    }
    wave_best(v, i);
    float* sv = s_val[round & 1];                   // two sets in turn: one barrier a round
    int* si = s_idx[round & 1];
    if (lane == 0) { sv[w] = v; si[w] = i; }
    __syncthreads();
    float bv = sv[0];
    int bi = si[0];
#pragma unroll
    for (int x = 1; x < 4; ++x)
      if (better(sv[x], si[x], bv, bi)) { bv = sv[x]; bi = si[x]; }
    chunk = (bv == -INFINITY) ? -1 : bi;
    if (chunk < 0) break;
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (tid + 256 * q == chunk) mine[q] = -INFINITY;
  }
  if (blockIdx.z == 0 && tid == 0) a.chunk_id[b * KMAX + k] = chunk;
  if (chunk < 0) return;                            // fewer than k+1 chunks hold anything
  // ---- its logits: four vocabulary rows at a time, so that their loads are in flight together (every row keeps its own
  // accumulation order: the logits are those of one row after the other)
  const T* x = reinterpret_cast<const T*>(a.nf) + (size_t)r * a.d;
  float* logits = a.logits + ((size_t)b * KMAX + k) * 128;
  const int rows = 128 / (int)gridDim.z;
  for (int i = blockIdx.z * rows + w * 4; i < (int)(blockIdx.z + 1) * rows; i += 16) {
    const int v0 = chunk * 128 + i;
    float l[4];
    if (v0 + 3 < a.V) {
      dot_rows4<T>(x, reinterpret_cast<const T*>(a.w_vocab) + (size_t)v0 * a.d, a.d, lane, l);
#pragma unroll
      for (int u = 0; u < 4; ++u) l[u] *= a.scale;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        l[u] = -INFINITY;
        if (v0 + u < a.V) l[u] = dot_row<T>(x, reinterpret_cast<const T*>(a.w_vocab) + (size_t)(v0 + u) * a.d, a.d, lane) * a.scale;
      }
    }
    if (lane == 0) *reinterpret_cast<f32x4*>(logits + i) = f32x4{l[0], l[1], l[2], l[3]};
  }
}

// one workgroup per position, whole vocabulary; candidates go to slot k = 0
template <typename T>
__global__ __launch_bounds__(256) void topk_full_kernel(HeadTopkArgs a) {
  __shared__ float s_v[4][KMAX];
  __shared__ int s_i[4][KMAX];
  const int b = blockIdx.x;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int node = a.result ? a.result->node : a.node;
  float* cv = a.cand_val + (size_t)b * KMAX * KMAX;
  int32_t* ci = a.cand_idx + (size_t)b * KMAX * KMAX;
  for (int e = tid; e < KMAX * KMAX; e += 256) { cv[e] = -INFINITY; ci[e] = -1; }
  const int r = (node >= 0 && node < a.G) ? find_row(a.row_idx, min(*a.count, a.G * a.B), node * a.B + b) : -1;
  if (r < 0) return;
  const T* x = reinterpret_cast<const T*>(a.nf) + (size_t)r * a.d;
  float tv[KMAX];
  int ti[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) { tv[j] = -INFINITY; ti[j] = 0x7fffffff; }
  for (int v = w; v < a.V; v += 4) {                // increasing token id per wavefront
    float l = dot_row<T>(x, reinterpret_cast<const T*>(a.w_vocab) + (size_t)v * a.d, a.d, lane) * a.scale;
    int li = v;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {               // sorted insertion: swap down while the newcomer is better
      if (better(l, li, tv[j], ti[j])) {
        const float fv = tv[j]; const int fi = ti[j];
        tv[j] = l; ti[j] = li;
        l = fv; li = fi;
      }
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) { s_v[w][j] = tv[j]; s_i[w][j] = ti[j]; }
  }
  __syncthreads();
  if (tid == 0) {
    int pos[4] = {0, 0, 0, 0};
    for (int j = 0; j < a.K; ++j) {                 // merge of four sorted lists
      int bw = -1;
      for (int x2 = 0; x2 < 4; ++x2) {
        if (pos[x2] >= KMAX) continue;
        if (bw < 0 || better(s_v[x2][pos[x2]], s_i[x2][pos[x2]], s_v[bw][pos[bw]], s_i[bw][pos[bw]])) bw = x2;
      }
      const float v = s_v[bw][pos[bw]];
      cv[j] = v;
      ci[j] = (v == -INFINITY) ? -1 : s_i[bw][pos[bw]];
      ++pos[bw];
    }
  }
}

// CHUNKS: the candidates are the logits of the row's K best chunks; otherwise the K best of the whole vocabulary.  A wavefront a
// chunk finds the chunk's best, then the first takes the best of those: 2 (K - 1) rounds of a wavefront's best with one or two
// candidates a lane.  (One wavefront with sixteen candidates a lane is a chain of comparisons: K = 8 13 - 19 us, 7 - 10 so.)
template <bool CHUNKS>
__global__ __launch_bounds__(64 * KMAX) void topk_merge_kernel(HeadTopkArgs a) {
  __shared__ float s_v[KMAX][KMAX];
  __shared__ int s_i[KMAX][KMAX];
  const int b = blockIdx.x, lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int node = a.result ? a.result->node : a.node;
  int32_t* ot = a.out_tokens + (size_t)b * a.K;
  float* op = a.out_probs + (size_t)b * a.K;
  const bool node_ok = node >= 0 && node < a.G;
  const int f = node_ok ? node * a.B + b : 0;
  const int r = node_ok ? find_row(a.row_idx, min(*a.count, a.G * a.B), f) : -1;
  if (r < 0) {                                      // not masked: nothing to draft here
    if (w == 0 && lane < a.K) { ot[lane] = node_ok ? a.tokens[f] : -1; op[lane] = 0.f; }
    return;
  }
  const TopPartial top = a.row_top[r];
  // Column 0 is the head's own argmax with the confidence it reported, whatever the recomputed candidates say
  // (their logits are summed in another order, so on a near-tie the head's token could otherwise drop out of its
  // chunk's K best, or come second).  The other K-1 places go to the best candidates other than that token; a
  // candidate whose recomputed logit exceeds the head's top logit is held at it, so probabilities never increase
  // along a row.
  constexpr int NONE = 0x7fffffff;                  // of value -inf
  float v = -INFINITY;
  int i = NONE;
  if (CHUNKS) {
    float cv[2];
    int ci[2];
    const int chunk = a.chunk_id[b * KMAX + w];     // uniform
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = lane + 64 * q;
      cv[q] = chunk >= 0 ? a.logits[((size_t)b * KMAX + w) * 128 + e] : -INFINITY;
      ci[q] = chunk * 128 + e;
      if (chunk < 0 || ci[q] == top.idx) { cv[q] = -INFINITY; ci[q] = NONE; }
    }
    for (int j = 1; j < a.K; ++j) {
      float bv = cv[0];
      int bi = ci[0];
      keep_better(bv, bi, cv[1], ci[1]);
      wave_best(bv, bi);
      if (lane == 0) { s_v[w][j] = bv; s_i[w][j] = bv == -INFINITY ? NONE : bi; }
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (ci[q] == bi) { cv[q] = -INFINITY; ci[q] = NONE; }
    }
    __syncthreads();
    if (w > 0) return;
    const int k = lane / KMAX, j = lane % KMAX;
    if (k < a.K && j > 0 && j < a.K) { v = s_v[k][j]; i = s_i[k][j]; }
  } else if (lane < a.K) {
    i = a.cand_idx[(size_t)b * KMAX * KMAX + lane];
    v = a.cand_val[(size_t)b * KMAX * KMAX + lane];
    if (i < 0 || i == top.idx) { v = -INFINITY; i = NONE; }
  }
  if (lane == 0) { ot[0] = top.idx; op[0] = 1.0f / top.s; }
  for (int j = 1; j < a.K; ++j) {
    float bv = v;
    int bi = i;
    wave_best(bv, bi);
    const bool any = bv != -INFINITY;               // -inf: no candidate is left
    if (lane == 0) {
      ot[j] = any ? bi : -1;
      op[j] = any ? __expf(fminf(bv, top.m) - top.m) / top.s : 0.f;
    }
    if (i == bi) { v = -INFINITY; i = NONE; }
  }
}

}  // namespace

hipError_t launch_head_topk(const HeadTopkArgs& a, hipStream_t st) {
  if (a.K < 1 || a.K > KMAX || a.B < 1) return hipErrorInvalidValue;
  if (a.n_part > 0) {
    if (a.n_part > 2048 || a.dtype != SPIFFY_BF16 || a.d % 8 != 0) return hipErrorInvalidValue;
    topk_refine_kernel<bf16_t><<<dim3(a.B, a.K, refine_slices(a.B, a.K, a.d)), 256, 0, st>>>(a);
    topk_merge_kernel<true><<<a.B, 64 * a.K, 0, st>>>(a);
    return hipGetLastError();
  }
  if (a.dtype == SPIFFY_F32) {
    topk_full_kernel<float><<<a.B, 256, 0, st>>>(a);
  } else {
    if (a.d % 8 != 0) return hipErrorInvalidValue;
    topk_full_kernel<bf16_t><<<a.B, 256, 0, st>>>(a);
  }
  topk_merge_kernel<false><<<a.B, 64, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace spiffy
