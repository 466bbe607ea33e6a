// Shared device/host helpers for the gfx950 kernels (no entry points here).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/spiffy.h"

namespace spiffy {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return static_cast<float>(x); }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return static_cast<bf16_t>(x); }

// Reductions over the wavefront, distances 32, 16, .. 1 in turn, every lane gets the result.  The partner's value comes from
// vector instructions (swaps of 32- and 16-lane rows hold both values in one lane, then DPP permutations); __shfl_xor takes
// each through the LDS crossbar, some 60 cycles a step.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <typename Op>
__device__ __forceinline__ float reduce_32(float v, Op op) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <typename Op>
__device__ __forceinline__ float reduce_16(float v, Op op) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
  v = reduce_16(reduce_32(v, op), op);
  v = op(v, dpp_move<0x128>(v));                       // row_ror:8
  v = op(v, dpp_move<0x1B>(dpp_move<0x141>(v)));       // lane ^ 7, then lane ^ 3
  v = op(v, dpp_move<0x4E>(v));                        // quad_perm [2,3,0,1]
  return op(v, dpp_move<0xB1>(v));                     // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}

// Running summary of a set of logits: top value, its lowest index, runner-up value and
// sum of exp(l - top).  Merging two summaries is exact for (top, index) and stable for the sum.
struct Top {
  float m;   // top logit (-inf when empty)
  float m2;  // second logit (-inf when fewer than two)
  float s;   // sum exp(l - m)
  int idx;   // lowest index attaining m
};
__device__ __forceinline__ Top top_empty() { return Top{-INFINITY, -INFINITY, 0.f, 0x7fffffff}; }
__device__ __forceinline__ Top top_merge(const Top& a, const Top& b) {
  Top r;
  if (a.m > b.m || (a.m == b.m && a.idx <= b.idx)) {
    r.m = a.m; r.idx = a.idx; r.m2 = fmaxf(a.m2, b.m);
  } else {
    r.m = b.m; r.idx = b.idx; r.m2 = fmaxf(b.m2, a.m);
  }
  float sa = (a.m == -INFINITY) ? 0.f : a.s * __expf(a.m - r.m);
  float sb = (b.m == -INFINITY) ? 0.f : b.s * __expf(b.m - r.m);
  r.s = sa + sb;
  return r;
}
__device__ __forceinline__ Top top_shfl_xor(const Top& a, int o) {
  Top b;
  b.m = __shfl_xor(a.m, o, 64);
  b.m2 = __shfl_xor(a.m2, o, 64);
  b.s = __shfl_xor(a.s, o, 64);
  b.idx = __shfl_xor(a.idx, o, 64);
  return b;
}

// Per-row partial written by the LM-head kernels and merged by the combine kernel.
struct alignas(16) TopPartial {
  float m, m2, s;
  int idx;
};

// ---------------------------------------------------------------------------------------------
// launch parameter blocks (plain structs passed by value)
// ---------------------------------------------------------------------------------------------

// C[M,N] = A[M,K] * W^T where W is given as up to three row-major [N_i,K] segments laid side by
// side along N (q | k | v), or as a (gate, up) pair for the SwiGLU epilogue.
enum GemmEpi { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LMHEAD = 3, EPI_PARTIAL = 4, EPI_QKV = 5 };

// EPI_QKV (head_dim 128): rotary embedding of the q and k columns, scale of q, and the rows that also go to the cache.
// Row g of the whole product has table row g % B while g < rows, B + g - rows behind (rows that ride along with the states).
struct QkvArgs {
  const void* rope;     // [32][rope_rows] (cos, sin, cos, sin) of two neighbouring frequencies: a lane's neighbours are other rows
  int rope_rows;
  void *ck, *cv;        // cache [Hkv][ldp][128]; k and v of rows 0 .. n_head-1 go to cache rows dst_head .., of the rows
  int ldp;              // behind `rows` to dst_tail .. (dst_tail < 0: not)
  int row0, rows, B;    // row0: row of the whole product that is row 0 of this launch
  unsigned magic;       // ceil(2^32 / B): g / B = (g * magic) >> 32 for g, B < 65536 (B > 1)
  int n_head, dst_head, dst_tail;
  float q_scale;
};

struct GemmArgs {
  const void* A;        // [M,K]
  const void* W[3];     // segments, each [Nseg[i],K]; SWIGLU: W[0]=gate, W[1]=up, each [N,K]
  const void* bias[3];  // optional per-segment bias (fp32 math), NULL = none
  int Nseg[3];
  void* C;              // [M,N] (STORE/RESID/SWIGLU); LMHEAD: TopPartial [M, n_tiles_total]
  const void* R;        // residual [M,N] for EPI_RESID
  const int* M_dev;     // optional device row count (rows >= *M_dev are skipped), NULL = use M
  const int32_t* a_rows; // PARTIAL: optional row list, row r of the product reads row a_rows[r] of A (r < *M_dev)
  int M, N, K;
  int lda, ldc;
  int ldw;              // row stride of the weight segments in elements (0 = K, i.e. dense rows)
  float scale;          // LMHEAD: logit scale
  int ksplit;           // PARTIAL: number of K slices (C = fp32 [ksplit][Mz][N]); otherwise 1
  QkvArgs qkv;          // QKV only
  int Mz;               // PARTIAL: rows per K slice of C when only some of them are computed by this launch (0 = M)
};

// Rotary table: `rows` rows of `half` (cos, sin) pairs, rows 0 .. B-1 at positions pos0 .., rows B .. at tail_pos0 ...
// paired: [half / 2][rows][2] (lanes of the QKV projection's epilogue are rows), otherwise [rows][half].
struct RopeArgs {
  float2* tab;
  int rows, B, half, pos0, tail_pos0, paired;
  float base;
};
// entry i: angle in double, cos and sin rounded to float
__device__ __forceinline__ void rope_entry(const RopeArgs& a, int i) {
  const int f = a.paired ? 2 * (i / (2 * a.rows)) + i % 2 : i % a.half, b = a.paired ? (i / 2) % a.rows : i / a.half;
  const double inv_freq = pow((double)a.base, -(double)f / (double)a.half);
  const double ang = (double)(b < a.B ? a.pos0 + b : a.tail_pos0 + b - a.B) * inv_freq;
  a.tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}

// Workgroup ids are handed to the 8 XCDs round-robin (id % 8).  Map id -> logical index so that every
// XCD owns one contiguous range of logical indices (XCD x owns ids x, x+8, ...), for any total.
__device__ __forceinline__ int xcd_contiguous(int id, int total) {
  const int x = id & 7, j = id >> 3;
  const int q = total >> 3, r = total & 7;
  return x * q + (x < r ? x : r) + j;
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Raise a kernel's dynamic LDS limit once per device: `done` holds one bit per device id.  Safe from several host
// threads (setting the attribute twice is harmless).
inline hipError_t allow_dynamic_lds(const void* kernel, int bytes, std::atomic<unsigned long long>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const unsigned long long bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace spiffy
