// Small steps of every configuration (fp32 math, float or bf16 storage): embedding gather, RMSNorm, masked-row
// compaction, prefix-cache extension, the LM-head combine and the decision step (Alg. 1 steps 1-4).
#include "kernels.h"

namespace spiffy {

// ---------------------------------------------------------------------------------------------
// row gather of two matrices with one row list: a_out[r,:] = a[row_idx[r],:], b_out[r,:] = b[row_idx[r],:]
// for r < *count (the masked rows of the last layer: attention output and residual stream)
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gather_rows2_kernel(const uint4* __restrict__ a, int a16, const uint4* __restrict__ b,
                                                           int b16, const int32_t* __restrict__ row_idx,
                                                           const int32_t* __restrict__ count, uint4* __restrict__ a_out,
                                                           uint4* __restrict__ b_out) {
  const int r = blockIdx.x;
  if (r >= *count) return;
  const size_t src = (size_t)row_idx[r];
  for (int i = threadIdx.x; i < a16; i += 256) a_out[(size_t)r * a16 + i] = a[src * a16 + i];
  for (int i = threadIdx.x; i < b16; i += 256) b_out[(size_t)r * b16 + i] = b[src * b16 + i];
}

// out[row_idx[r],:] = in[r,:] for r < *count
__global__ __launch_bounds__(256) void scatter_rows_kernel(const uint4* __restrict__ in, int n16, const int32_t* __restrict__ row_idx,
                                                           const int32_t* __restrict__ count, uint4* __restrict__ out) {
  const int r = blockIdx.x;
  if (r >= *count) return;
  const size_t dst = (size_t)row_idx[r];
  for (int i = threadIdx.x; i < n16; i += 256) out[dst * n16 + i] = in[(size_t)r * n16 + i];
}

hipError_t launch_scatter_rows(const void* in, size_t row_bytes, const int32_t* row_idx, const int32_t* count, int M,
                               void* out, hipStream_t st) {
  scatter_rows_kernel<<<M, 256, 0, st>>>((const uint4*)in, (int)(row_bytes / 16), row_idx, count, (uint4*)out);
  return hipGetLastError();
}

hipError_t launch_gather_rows2(const void* a, size_t a_row_bytes, const void* b, size_t b_row_bytes,
                               const int32_t* row_idx, const int32_t* count, int M, void* a_out, void* b_out,
                               hipStream_t st) {
  gather_rows2_kernel<<<M, 256, 0, st>>>((const uint4*)a, (int)(a_row_bytes / 16), (const uint4*)b, (int)(b_row_bytes / 16),
                                         row_idx, count, (uint4*)a_out, (uint4*)b_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// RMSNorm with optional row gather
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// row `src` of x, normalised, to row `r` of out: one workgroup, 16 bytes per thread per step; d * sizeof(T) is a multiple of
// 16 (checked by the host)
template <typename T>
__device__ __forceinline__ void rmsnorm_row(const T* __restrict__ x, const T* __restrict__ gain, float eps, int d, int src,
                                            int r, T* __restrict__ out, float* red) {
  constexpr int VEC = 16 / sizeof(T);
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  const vec_t* xr = reinterpret_cast<const vec_t*>(x + (size_t)src * d);
  const vec_t* gr = reinterpret_cast<const vec_t*>(gain);
  vec_t* o = reinterpret_cast<vec_t*>(out + (size_t)r * d);
  const int nv = d / VEC;
  float ss = 0.f;
  for (int i = threadIdx.x; i < nv; i += 256) {
    const vec_t v = xr[i];
#pragma unroll
    for (int e = 0; e < VEC; ++e) { const float f = to_f32(v[e]); ss += f * f; }
  }
  ss = block_sum_256(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int i = threadIdx.x; i < nv; i += 256) {
    const vec_t v = xr[i], g = gr[i];
    vec_t w;
#pragma unroll
    for (int e = 0; e < VEC; ++e) w[e] = from_f32<T>(to_f32(v[e]) * inv * to_f32(g[e]));
    o[i] = w;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const T* __restrict__ x, const T* __restrict__ gain, float eps,
                                                      int M, int d, const int32_t* __restrict__ row_idx,
                                                      const int32_t* __restrict__ n_rows_dev, T* __restrict__ out) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  const int n_rows = n_rows_dev ? *n_rows_dev : M;
  if (r >= n_rows) return;
  rmsnorm_row<T>(x, gain, eps, d, row_idx ? row_idx[r] : r, r, out, red);
}

// Masked-row list and normalised masked rows in one launch: workgroup m counts the masked rows before its own row.  The
// list alone took a launch of 2.0 - 4.6 us in front of this one; the counting reads M tokens per masked row from L2.
template <typename T>
__global__ __launch_bounds__(256) void masked_rmsnorm_kernel(const T* __restrict__ x, const T* __restrict__ gain, float eps,
                                                             int M, int d, const int32_t* __restrict__ tok,
                                                             const uint8_t* __restrict__ mask, int mask_id,
                                                             int32_t* __restrict__ row_idx, int32_t* __restrict__ count,
                                                             T* __restrict__ out) {
  __shared__ float red[4];
  __shared__ int before[4];
  const int m = blockIdx.x;
  auto masked = [&](int i) { return mask ? (mask[i] != 0) : (tok[i] == mask_id); };
  const bool mk = masked(m);
  if (!mk && m != M - 1) return;                   // the last row leaves the count, masked or not
  int c = 0;
  for (int i = threadIdx.x; i < m; i += 256) c += masked(i) ? 1 : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((threadIdx.x & 63) == 0) before[threadIdx.x >> 6] = c;
  __syncthreads();
  const int r = before[0] + before[1] + before[2] + before[3];
  if (threadIdx.x == 0) {
    if (mk) row_idx[r] = m;
    if (m == M - 1) *count = r + (mk ? 1 : 0);
  }
  if (mk) rmsnorm_row<T>(x, gain, eps, d, m, r, out, red);
}

hipError_t launch_rmsnorm(int dtype, const void* x, const void* gain, float eps, int M, int d,
                          const int32_t* row_idx, const int32_t* n_rows_dev, void* out, hipStream_t st) {
  if (dtype == SPIFFY_F32)
    rmsnorm_kernel<float><<<M, 256, 0, st>>>((const float*)x, (const float*)gain, eps, M, d, row_idx, n_rows_dev,
                                             (float*)out);
  else
    rmsnorm_kernel<bf16_t><<<M, 256, 0, st>>>((const bf16_t*)x, (const bf16_t*)gain, eps, M, d, row_idx,
                                              n_rows_dev, (bf16_t*)out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// masked-row compaction: row_idx[0..count) ascending, plus count (one workgroup)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void compact_rows(const int32_t* __restrict__ tok, const uint8_t* __restrict__ mask, int mask_id,
                                             int M, int32_t* __restrict__ row_idx, int32_t* __restrict__ count, int* cnt) {
  const int per = (M + 255) / 256;
  const int i0 = threadIdx.x * per, i1 = min(M, i0 + per);
  int c = 0;
  for (int i = i0; i < i1; ++i) c += mask ? (mask[i] != 0) : (tok[i] == mask_id);
  cnt[threadIdx.x] = c;
  __syncthreads();
  // exclusive scan by a simple doubling pass
  for (int o = 1; o < 256; o <<= 1) {
    const int v = (threadIdx.x >= o) ? cnt[threadIdx.x - o] : 0;
    __syncthreads();
    cnt[threadIdx.x] += v;
    __syncthreads();
  }
  int pos = cnt[threadIdx.x] - c;
  for (int i = i0; i < i1; ++i) {
    const bool mk = mask ? (mask[i] != 0) : (tok[i] == mask_id);
    if (mk) row_idx[pos++] = i;
  }
  if (threadIdx.x == 255) *count = cnt[255];
}

__global__ __launch_bounds__(256) void compact_rows_kernel(const int32_t* __restrict__ tok,
                                                           const uint8_t* __restrict__ mask, int mask_id, int M,
                                                           int32_t* __restrict__ row_idx, int32_t* __restrict__ count) {
  __shared__ int cnt[256];
  compact_rows(tok, mask, mask_id, M, row_idx, count, cnt);
}

hipError_t launch_compact_rows(const int32_t* tok, const uint8_t* mask, int mask_id, int M, int32_t* row_idx,
                               int32_t* count, hipStream_t st) {
  compact_rows_kernel<<<1, 256, 0, st>>>(tok, mask, mask_id, M, row_idx, count);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void rope_table_kernel(RopeArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < a.rows * a.half) rope_entry(a, i);
}

hipError_t launch_rope_table(const RopeArgs& a, hipStream_t st) {
  rope_table_kernel<<<cdiv(a.rows * a.half, 256), 256, 0, st>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Start of a step.  Embedding gather: out[m,:] = w[tok[m],:], rows M .. M+M2-1 from tok2; with a gain also n_out[m,:] =
// RMSNorm of that row, which the first layer starts from (a launch of its own took 2.9 - 4.2 us; the row is still in L1
// here).  Beside the rows, in workgroups of their own, what later kernels of the step need and nothing before them
// provides: the rotary table and the list of masked rows, which had launches of 4.7 us each.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(EmbedArgs a, int rope_blocks, int list_blocks) {
  __shared__ int cnt[256];
  int m = blockIdx.x;
  if (m < rope_blocks) {
    const int i = m * 256 + threadIdx.x;
    if (i < a.rope.rows * a.rope.half) rope_entry(a.rope, i);
    return;
  }
  m -= rope_blocks;
  if (m < list_blocks) {
    compact_rows(a.tok, nullptr, a.mask_id, a.M, a.rows, a.count, cnt);
    return;
  }
  m -= list_blocks;
  int t = m < a.M ? a.tok[m] : a.tok2[m - a.M];
  t = t < 0 ? 0 : (t >= a.V ? a.V - 1 : t);
  const T* w = reinterpret_cast<const T*>(a.w);
  const uint4* src = reinterpret_cast<const uint4*>(w + (size_t)t * a.d);
  uint4* dst = reinterpret_cast<uint4*>(reinterpret_cast<T*>(a.out) + (size_t)m * a.d);
  const int n16 = a.d * (int)sizeof(T) / 16;
  for (int i = threadIdx.x; i < n16; i += blockDim.x) dst[i] = src[i];
  if (a.gain)
    rmsnorm_row<T>(w, reinterpret_cast<const T*>(a.gain), a.eps, a.d, t, m, reinterpret_cast<T*>(a.n_out),
                   reinterpret_cast<float*>(cnt));
}

hipError_t launch_embed(int dtype, const EmbedArgs& a, hipStream_t st) {
  const int rope = a.rope.tab ? cdiv(a.rope.rows * a.rope.half, 256) : 0, list = a.rows ? 1 : 0;
  const int grid = rope + list + a.M + a.M2;
  if (dtype == SPIFFY_F32) embed_kernel<float><<<grid, 256, 0, st>>>(a, rope, list);
  else embed_kernel<bf16_t><<<grid, 256, 0, st>>>(a, rope, list);
  return hipGetLastError();
}

// The counting grows with M * M and the list's launch does not.  The head, 256 tokens of vocabulary, width 1024 in bf16 / 4096 in bf16
// / 1024 in fp32, every row masked, us with one launch and with two: 2048 rows 35.8, 38.7 / 73.0, 78.6 / 57.3, 60.9; 8192 rows 57.2, 61.8
// / 98.9, 105.8 / 114, 120; 16384 rows 99.1, 80.6 / 160, 149 / 229, 216.
hipError_t launch_masked_rmsnorm(int dtype, const void* x, const void* gain, float eps, int M, int d, const int32_t* tok,
                                 const uint8_t* mask, int mask_id, int32_t* row_idx, int32_t* count, void* out,
                                 hipStream_t st) {
  if (M > 8192) {
    const hipError_t e = launch_compact_rows(tok, mask, mask_id, M, row_idx, count, st);
    return e != hipSuccess ? e : launch_rmsnorm(dtype, x, gain, eps, M, d, row_idx, count, out, st);
  }
  if (dtype == SPIFFY_F32)
    masked_rmsnorm_kernel<float><<<M, 256, 0, st>>>((const float*)x, (const float*)gain, eps, M, d, tok, mask, mask_id,
                                                    row_idx, count, (float*)out);
  else
    masked_rmsnorm_kernel<bf16_t><<<M, 256, 0, st>>>((const bf16_t*)x, (const bf16_t*)gain, eps, M, d, tok, mask, mask_id,
                                                     row_idx, count, (bf16_t*)out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// prefix-cache extension: one thread per (token b, kv head, frequency f)
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void kv_append_kernel(const T* __restrict__ qkv, int Hq, int Hkv, int hd, int B,
                                                        int pos0, float base, T* __restrict__ ck, T* __restrict__ cv,
                                                        int P, int ldp, int B0, int skip) {
  const int half = hd / 2;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= B * Hkv * half) return;
  const int f = i % half, kvh = (i / half) % Hkv, b = i / (half * Hkv);
  const int ld = (Hq + 2 * Hkv) * hd;
  const int src = b < B0 ? b : b + skip;      // the rows may come in two runs: B0 rows, `skip` rows that are not appended, the rest
  const T* kr = qkv + (size_t)src * ld + (Hq + kvh) * hd;
  const T* vr = qkv + (size_t)src * ld + (Hq + Hkv + kvh) * hd;
  // same values as the rotary table of the attention kernel: angle in double, cos / sin rounded to float
  const double inv_freq = pow((double)base, -2.0 * (double)f / (double)hd);
  const double ang = (double)(pos0 + b) * inv_freq;
  const float c = (float)cos(ang), s = (float)sin(ang);
  const float x1 = to_f32(kr[f]), x2 = to_f32(kr[f + half]);
  T* kd = ck + ((size_t)kvh * ldp + P + b) * hd;
  T* vd = cv + ((size_t)kvh * ldp + P + b) * hd;
  kd[f] = from_f32<T>(x1 * c - x2 * s);
  kd[f + half] = from_f32<T>(x2 * c + x1 * s);
  vd[f] = vr[f];
  vd[f + half] = vr[f + half];
}

hipError_t launch_kv_append(int dtype, const void* qkv, int Hq, int Hkv, int hd, int B, int pos0, float rope_base,
                            void* cache_k, void* cache_v, int P, int ldp, hipStream_t st, int B0, int skip) {
  if (B0 <= 0) { B0 = B; skip = 0; }
  const int n = B * Hkv * (hd / 2);
  if (dtype == SPIFFY_F32)
    kv_append_kernel<float><<<cdiv(n, 256), 256, 0, st>>>((const float*)qkv, Hq, Hkv, hd, B, pos0, rope_base,
                                                          (float*)cache_k, (float*)cache_v, P, ldp, B0, skip);
  else
    kv_append_kernel<bf16_t><<<cdiv(n, 256), 256, 0, st>>>((const bf16_t*)qkv, Hq, Hkv, hd, B, pos0, rope_base,
                                                           (bf16_t*)cache_k, (bf16_t*)cache_v, P, ldp, B0, skip);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// merge the per-tile partial summaries part[n_part][m_cap] of each row; lanes run along rows so
// the reads are coalesced, four wavefronts split the partials of the same 64 rows.  blockIdx.y
// selects a slice of the partials (two-level merge when there are many): out is [gridDim.y][m_cap].
__global__ __launch_bounds__(256) void lmhead_combine_kernel(const TopPartial* __restrict__ part, int n_part,
                                                             int m_cap, const int32_t* __restrict__ count,
                                                             TopPartial* __restrict__ out) {
  __shared__ TopPartial sh[4][64];
  const int n = *count;
  const int r0 = blockIdx.x * 64;
  if (r0 >= n) return;
  const int per = (n_part + gridDim.y - 1) / gridDim.y;
  const int p0 = blockIdx.y * per, p1 = min(n_part, p0 + per);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = r0 + lane;
  Top t = top_empty();
  if (r < n) {
    // sixteen loads in flight: one at a time the loop was a chain of memory latencies (11.3 us for 32 rows of 988 summaries,
    // 5.0 like this); the merges keep their order
    constexpr int NB = 16;
    for (int i0 = p0 + w; i0 < p1; i0 += 4 * NB) {
      TopPartial p[NB];
#pragma unroll
      for (int k = 0; k < NB; ++k)
        if (i0 + 4 * k < p1) p[k] = part[(size_t)(i0 + 4 * k) * m_cap + r];
#pragma unroll
      for (int k = 0; k < NB; ++k)
        if (i0 + 4 * k < p1) t = top_merge(t, Top{p[k].m, p[k].m2, p[k].s, p[k].idx});
    }
  }
  sh[w][lane] = TopPartial{t.m, t.m2, t.s, t.idx};
  __syncthreads();
  if (w == 0 && r < n) {
    Top a = top_empty();
    for (int i = 0; i < 4; ++i) a = top_merge(a, Top{sh[i][lane].m, sh[i][lane].m2, sh[i][lane].s, sh[i][lane].idx});
    out[(size_t)blockIdx.y * m_cap + r] = TopPartial{a.m, a.m2, a.s, a.idx};
  }
}

hipError_t launch_lmhead_combine(const TopPartial* part, int n_part, int m_cap, const int32_t* count, int M,
                                 TopPartial* tmp, TopPartial* row_top, int* n_sums, hipStream_t st) {
  const int slices = kLmheadCombineSlices;
  *n_sums = n_part > 2 * slices && tmp ? slices : 1;
  lmhead_combine_kernel<<<dim3(cdiv(M, 64), *n_sums), 256, 0, st>>>(part, n_part, m_cap, count,
                                                                    *n_sums > 1 ? tmp : row_top);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// decisions per state (Alg. 1 steps 2-4 + threshold rule): one wavefront per state g.  A row's summary comes as
// kLmheadCombineSlices parts (SLICED), merged here: a state's rows are few and its lanes read them side by side, so the
// merge costs one round of loads where a launch of its own took 4 us (3.8 - 4.8 by the kernel trace, 32 to 128 rows).
// ---------------------------------------------------------------------------------------------
template <bool SLICED>
__global__ __launch_bounds__(64) void head_finalize_kernel(const TopPartial* __restrict__ sums, int m_cap,
                                                           TopPartial* __restrict__ row_top,
                                                           const int32_t* __restrict__ row_idx,
                                                           const int32_t* __restrict__ count,
                                                           const int32_t* __restrict__ tok,
                                                           const uint8_t* __restrict__ mask, int mask_id, int B,
                                                           float threshold, int force_one,
                                                           int32_t* __restrict__ argmax, float* __restrict__ conf,
                                                           uint8_t* __restrict__ unmask, float* __restrict__ margin,
                                                           int32_t* __restrict__ target) {
  const int g = blockIdx.x;
  const int lane = threadIdx.x;
  const int n = *count;
  // first compacted row belonging to state g: lower bound of g*B in the ascending row list
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (row_idx[mid] < g * B) lo = mid + 1; else hi = mid;
  }
  float best_c = -1.f;     // highest confidence among this lane's masked positions
  int best_b = 0x7fffffff, best_am = 0;
  bool any_pass = false;
  int base = lo;
  for (int b0 = 0; b0 < B; b0 += 64) {
    const int b = b0 + lane;
    const bool in = b < B;
    const int m = g * B + (in ? b : 0);
    const int t = in ? tok[m] : 0;
    const bool mk = in && (mask ? (mask[m] != 0) : (t == mask_id));
    const unsigned long long bal = __ballot(mk);
    const int r = base + __popcll(bal & ((1ull << lane) - 1ull));
    base += __popcll(bal);
    if (in) {
      int am = t;
      float cf = 0.f, mg = INFINITY;
      uint8_t um = 0;
      if (mk) {
        TopPartial p;
        if constexpr (SLICED) {                  // four chains, then their sum: the order of lmhead_combine_kernel
          constexpr int N = kLmheadCombineSlices;
          TopPartial part[N];
#pragma unroll
          for (int i = 0; i < N; ++i) part[i] = sums[(size_t)i * m_cap + r];
          Top a = top_empty();
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            Top t4 = top_empty();
#pragma unroll
            for (int i = w; i < N; i += 4) t4 = top_merge(t4, Top{part[i].m, part[i].m2, part[i].s, part[i].idx});
            a = top_merge(a, t4);
          }
          p = TopPartial{a.m, a.m2, a.s, a.idx};
          row_top[r] = p;                        // the drafting source reads it
        } else {
          p = sums[r];
        }
        am = p.idx;
        cf = 1.0f / p.s;
        mg = p.m - p.m2;
        um = cf > threshold ? 1 : 0;
        if (um) any_pass = true;
        if (cf > best_c) { best_c = cf; best_b = b; best_am = am; }
      }
      argmax[m] = am;
      conf[m] = cf;
      unmask[m] = um;
      if (margin) margin[m] = mg;
      if (target) target[m] = um ? am : t;
    }
  }
  const bool any = __ballot(any_pass) != 0ull;
  if (force_one && !any) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float oc = __shfl_xor(best_c, o, 64);
      const int ob = __shfl_xor(best_b, o, 64);
      const int oa = __shfl_xor(best_am, o, 64);
      if (oc > best_c || (oc == best_c && ob < best_b)) { best_c = oc; best_b = ob; best_am = oa; }
    }
    if (best_c >= 0.f && lane == (best_b & 63)) {   // the lane that wrote this position rewrites it
      const int m = g * B + best_b;
      unmask[m] = 1;
      if (target) target[m] = best_am;
    }
  }
}

hipError_t launch_head_finalize(const TopPartial* tmp, int n_sums, int m_cap, TopPartial* row_top,
                                const int32_t* row_idx, const int32_t* count,
                                const int32_t* tok, const uint8_t* mask, int mask_id, int G, int B, float threshold,
                                int force_one, int32_t* argmax, float* conf, uint8_t* unmask, float* margin,
                                int32_t* target, hipStream_t st) {
  if (n_sums > 1)
    head_finalize_kernel<true><<<G, 64, 0, st>>>(tmp, m_cap, row_top, row_idx, count, tok, mask, mask_id, B, threshold,
                                                 force_one, argmax, conf, unmask, margin, target);
  else
    head_finalize_kernel<false><<<G, 64, 0, st>>>(row_top, m_cap, nullptr, row_idx, count, tok, mask, mask_id, B,
                                                  threshold, force_one, argmax, conf, unmask, margin, target);
  return hipGetLastError();
}

}  // namespace spiffy
