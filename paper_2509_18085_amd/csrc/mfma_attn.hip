// Shared-prefix block attention for gfx950 (bf16 MFMA, head_dim 128).
//
// Every one of the G states attends to the same P cached keys and to its own B keys only
// (Fig. 4: a draft block sees the true context and itself; Sec. 3.1 prefix caching).  The mask is
// never built: the prefix part is dense and shared, the own-block part is the block diagonal of
// the (G*B) x (G*B) score matrix.
//
// Work split: one workgroup = (query head, 128 consecutive query rows, one split of the prefix).
// A prefix K/V tile of 64 keys is staged in LDS once and used by all 128 query rows (4 states of
// 32 tokens, or 32 states of 4); workgroups of the same head run next to each other on one XCD
// so the tile comes from HBM once and from L2 afterwards.  The number of prefix splits depends on
// P only, so a row's arithmetic does not depend on G.  With few states (fewer such workgroups than CUs) a
// workgroup owns 96, 64 or 32 of the 128 rows instead and the other wavefront pairs only move data: more CUs
// stream, nothing else changes.  A step that carries a second group of rows (the recomputed suffix of a
// full-sequence model, or the block being committed) runs both attention problems in one launch.
//
// Everything the workgroup reads travels global -> LDS directly as whole 256-byte rows (LDS-DMA loads, no
// registers): the Q rows, the own-block K/V rows and prefix tiles 0 and 1 at the start, later tiles into rings of
// NSTAGE stages for K and V, up to NSTAGE-1 tiles ahead of the MFMAs, one barrier per tile.  Rows keep their [row][hd]
// layout in LDS, 16-byte chunks permuted per row so that fragment reads are conflict-free:
//   Q / K row r: chunk c sits at position c ^ (r & 15)      (16-byte reads of one chunk per lane)
//   V row r: 64-byte unit u sits at position u ^ (r & 3)    (transposing 8-byte reads, below)
// What bounds the loop is the instruction stream of a SIMD's two wavefronts: 16 matrix instructions a tile and
// wavefront (512 cycles), whose shadow holds the exponentials but not much more, and the vector instructions around
// them.  Those are kept to what the softmax needs:
//   * the reference m of the online softmax follows the running maximum only when that is more than 8 ahead; the rescale
//     factor and its multiplies sit in a branch that is rarely taken;
//   * fragment addresses are loop invariant up to one add per two tiles (the stage is an immediate offset: K and V have
//     rings of their own, so two stages lie within its 64 KB); transfers use a scalar base and a constant lane offset;
//   * the score MFMAs of tile t+1 are issued between the exponentials of tile t.
// With both the kernel holds its state in 208 - 246 registers, nothing in scratch (before: 15 - 75 registers spilled).
// Measured, us: one or four states of 32 tokens behind 1024 rows 22.3 -> 16.3, 32 states 37.4 -> 31.2, 24 states of 28 heads
// behind 2048 rows 48.0 -> 41.1, 256 rows behind 8192 50.3 -> 45.2; 264 rows of blocks of 24 (144 workgroups of 32
// query rows where 48 of 128 ran) 34 -> 18.
//
// Eight wavefronts per workgroup: wavefront pair p owns query rows 32p..32p+31, and the two wavefronts
// of a pair split every 64-key tile between them (32 keys each), each keeping its own running
// (max, sum, O); the pair is merged through LDS at the end.  Two wavefronts per SIMD let the softmax
// arithmetic of one overlap the MFMAs of the other.
//
// Per wavefront (32 query rows x 32 keys of a tile) everything is kept "query per lane":
//   S^T = K Q^T    A operand = K rows from LDS, B operand = Q in registers
//                  -> lane (q, half) holds 16 of the 32 keys of a sub-tile for its query q
//   online softmax max / sum are reductions over the lane's own registers plus one half swap
//   O^T = V^T P^T  A operand = V^T, read from the row-major V tile with the transposing LDS read
//                  (ds_read_b64_tr_b16: in every group of 16 lanes, lane 4q+c receives element c of the
//                  8-byte pieces addressed by lanes q, q+4, q+8, q+12), B operand = P^T straight from
//                  the S^T accumulators (no trip through LDS); the rescale factor is per lane.
// Own-block keys (the block diagonal) come first, handled by the last prefix split: they always go to the
// wavefront of a pair that takes the first key half, in groups of 32 rows that are counted the same way however many query
// rows a workgroup owns, so a state's arithmetic does not depend on that; the mask is applied per element (any B works).
// Queries and keys arrive rotated (positions pos0..pos0+B-1 for every state, Sec. 4.3), queries also scaled by
// log2(e)/sqrt(128): the QKV projection's epilogue does both, in fp32 on the values rounded to bf16.
#include <type_traits>

#include "kernels.h"

namespace spiffy {

namespace {

constexpr int HD = 128;
constexpr int KTILE = 64;
constexpr int QTILE = 128;
constexpr int NSTAGE = 4;
constexpr int STAGE_BYTES = KTILE * HD * 2;               // one K or V tile: 16 KB
constexpr int V_RING = NSTAGE * STAGE_BYTES;              // K ring, V ring, then 128 own-block K rows
constexpr int OWN_K = 2 * NSTAGE * STAGE_BYTES;
constexpr int Q_ROWS = 2 * STAGE_BYTES;                   // before the loop: Q in K stages 2 and 3,
constexpr int OWN_V = V_RING + 2 * STAGE_BYTES;           // 128 own-block V rows in V stages 2 and 3
constexpr int SPLIT_KEYS = 2048;
constexpr size_t kAttnSmem = OWN_K + 2 * STAGE_BYTES;     // 163,840 B

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(3))) bf16x4* lds_bf16x4_ptr_t;
typedef const __attribute__((address_space(3))) bf16x8* lds_bf16x8_ptr_t;

constexpr int NT = 512;   // threads per workgroup
constexpr int DMA_PER_TILE = 4;   // LDS-DMA loads per thread per prefix tile (2 for K, 2 for V)

template <int N>
__device__ __forceinline__ void wait_vmcnt() {   // vmcnt <= N; lgkmcnt / expcnt untouched
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// position (in 16-byte chunks) of chunk c of row r inside the LDS tiles
__device__ __forceinline__ int k_pos(int r, int c) { return c ^ (r & 15); }
__device__ __forceinline__ int v_pos(int r, int c) { return c ^ ((r & 3) << 2); }

// Addresses are 32-bit LDS byte offsets: the base of a ring (or of own-block rows) plus a per-lane part that never changes.
struct WaveState {
  bf16x8 qf[8];     // Q^T fragments: hd = 16*kk + 8*half + e
  f32x16 o[4];      // O^T accumulators: hd = 32*n + 8*(v/4) + 4*half + v%4, query = lane%32
  float m_run, l_run;
};

// max of a value and its partner 32 lanes away, without a trip through LDS: after the swap one result
// holds the low half's values in both halves, the other the high half's
__device__ __forceinline__ float max_with_other_half(float x) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Reference value m of the online softmax (probabilities are exp2(s - m), log2 domain).  It only follows the running
// maximum when that has moved by more than 8: until then exp2(s - m) stays below 2^8, which bf16 and the fp32 sums
// hold as well as values below 1, and a reference that stays put needs no rescale of O and l (the factor is exactly
// 1 and the 64 multiplies are skipped).  The choice is made per query, so a row's arithmetic does not depend on the
// rows that share its wavefront; (m, l, O) stay consistent and every later merge weighs partials by exp2(m - max m).
// Returns the factor of l; O is rescaled here, in place (the multiplies are opaque to the compiler so that the rarely
// taken branch around them does not cost a copy of the 64 accumulator registers on every tile).  The compiler does not see
// what the assembly reads: each accumulator's first multiply waits out the matrix instruction that may have written it (at most
// 19 wait states, here 24), and the last is followed by the two that a matrix instruction reading it could need.
__device__ __forceinline__ float follow_maximum(WaveState& w, float tile_max) {
  const float m_cand = fmaxf(w.m_run, tile_max);
  const float m_new = (m_cand - w.m_run > 8.0f) ? m_cand : w.m_run;     // first tile: m_run = -inf, the difference is +inf
  float alpha = 1.f;
  if (__builtin_amdgcn_ballot_w64(m_new != w.m_run) != 0) {
    alpha = (w.m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(w.m_run - m_new);
    w.m_run = m_new;
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float x = w.o[n][v];
        if (v == 0) asm volatile("s_nop 15\n\ts_nop 7\n\tv_mul_f32 %0, %1, %0" : "+v"(x) : "v"(alpha));
        else asm volatile("v_mul_f32 %0, %1, %0" : "+v"(x) : "v"(alpha));
        w.o[n][v] = x;
      }
    asm volatile("s_nop 1");
  }
  return alpha;
}

// The lane's fragment addresses for 32 rows starting at row `row0` (a multiple of 32) of a tile at LDS address `base`
struct KAddr { unsigned a[8]; };      // K / Q: chunk 2*kk + half of row row0 + lane%32
struct VAddr { unsigned a[4]; };      // V^T, hd block n
__device__ __forceinline__ KAddr k_addr(unsigned base, int row0, int lane) {
  KAddr k;
  const int row = row0 + (lane & 31), hh = lane >> 5;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) k.a[kk] = base + row * (HD * 2) + k_pos(row, 2 * kk + hh) * 16;
  return k;
}
// lane j of a 16-lane group addresses key (j / 4) of its 4-key run, hd block 4 * (j % 4) of the group's 16 rows; the
// transposing read hands lane 4q+c the 4 keys of hd row 4q+c
__device__ __forceinline__ VAddr v_addr(unsigned base, int row0, int lane) {
  VAddr k;
  const int g = lane >> 4, j = lane & 15;
  const int vkey = row0 + 4 * (g >> 1) + (j >> 2);     // + 16*k2 + 8*eh, which keep (key & 3)
#pragma unroll
  for (int n = 0; n < 4; ++n) k.a[n] = base + vkey * (HD * 2) + (16 * (g & 1) + 4 * (j & 3)) * 2 + (n ^ (vkey & 3)) * 64;
  return k;
}
template <int OFF>
__device__ __forceinline__ bf16x8 k_frag(const KAddr& k, int kk) { return *(lds_bf16x8_ptr_t)(size_t)(k.a[kk] + OFF); }
template <int OFF>
__device__ __forceinline__ bf16x4 v_frag(const VAddr& k, int n, int k2, int eh) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr_t)(size_t)(k.a[n] + OFF + (16 * k2 + 8 * eh) * (HD * 2)));
}

// S^T of 32 keys: 8 MFMAs
template <int OFF>
__device__ __forceinline__ void scores(const WaveState& w, f32x16& s, const KAddr& ka) {
#pragma unroll
  for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag<OFF>(ka, kk), w.qf[kk], s, 0, 0, 0);
}

// Online-softmax update and O += P V for 32 keys whose scores are in registers and of which `valid(key)` says which count
template <typename ValidFn>
__device__ __forceinline__ void finish_masked(WaveState& w, f32x16& s, const VAddr& va, int lane, ValidFn valid) {
  const int hh = lane >> 5;
  float tmax = -INFINITY;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    if (!valid(8 * (v >> 2) + 4 * hh + (v & 3))) s[v] = -INFINITY;
    tmax = fmaxf(tmax, s[v]);
  }
  const float alpha = follow_maximum(w, max_with_other_half(tmax));
  const float m = (w.m_run == -INFINITY) ? 0.f : w.m_run;      // no valid key yet: every s is -inf
  bf16x8 pf[2];
  float psum = 0.f;
  const bf16x2 ones = {static_cast<bf16_t>(1.0f), static_cast<bf16_t>(1.0f)};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    f32x2 e;
    e[0] = __builtin_amdgcn_exp2f(s[2 * i] - m);
    e[1] = __builtin_amdgcn_exp2f(s[2 * i + 1] - m);
    const bf16x2 pb = __builtin_convertvector(e, bf16x2);
    psum = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, psum, false);
    pf[i >> 2][(2 * i) & 7] = pb[0];
    pf[i >> 2][(2 * i + 1) & 7] = pb[1];
  }
  w.l_run = w.l_run * alpha + psum;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const bf16x8 vf = __builtin_shufflevector(v_frag<0>(va, n, k2, 0), v_frag<0>(va, n, k2, 1), 0, 1, 2, 3, 4, 5, 6, 7);
      w.o[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[k2], w.o[n], 0, 0, 0);
    }
}

// One step of the software pipeline over full prefix tiles: the online-softmax arithmetic on the scores
// `s` of tile t runs between the score MFMAs of tile t+1 (K at ka + KOFF, result in `sn`),
// then O += P V for tile t (V at va + VOFF).
template <int KOFF, int VOFF>
__device__ __forceinline__ void pipe_step(WaveState& w, f32x16& s, f32x16& sn, const KAddr& ka, const VAddr& va) {
  bf16x8 kf[8];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) kf[kk] = k_frag<KOFF>(ka, kk);
  float tmax = s[0];
#pragma unroll
  for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
  const float alpha = follow_maximum(w, max_with_other_half(tmax));     // a full tile has no masked score: m_run is finite now
  const float m = w.m_run;
#pragma unroll
  for (int v = 0; v < 16; ++v) sn[v] = 0.f;
  bf16x8 pf[2];
  bf16x4 vlo[8], vhi[8];
  float psum = 0.f;
  const bf16x2 ones = {static_cast<bf16_t>(1.0f), static_cast<bf16_t>(1.0f)};
  __builtin_amdgcn_sched_barrier(0);   // K fragment reads and the maximum stay above this line
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], w.qf[i], sn, 0, 0, 0);
    f32x2 e;
    e[0] = __builtin_amdgcn_exp2f(s[2 * i] - m);
    e[1] = __builtin_amdgcn_exp2f(s[2 * i + 1] - m);
    const bf16x2 pb = __builtin_convertvector(e, bf16x2);
    psum = __builtin_amdgcn_fdot2_f32_bf16(pb, ones, psum, false);
    pf[i >> 2][(2 * i) & 7] = pb[0];
    pf[i >> 2][(2 * i + 1) & 7] = pb[1];
    vlo[i] = v_frag<VOFF>(va, i & 3, i >> 2, 0);      // V^T fragment i: key step i / 4, hd block i % 4
    vhi[i] = v_frag<VOFF>(va, i & 3, i >> 2, 1);
  }
  // issue order for the loop above: per score MFMA two exponentials with their subtract / convert / sum and two V fragment reads
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
  }
  w.l_run = w.l_run * alpha + psum;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bf16x8 vf = __builtin_shufflevector(vlo[i], vhi[i], 0, 1, 2, 3, 4, 5, 6, 7);
    w.o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[i >> 2], w.o[i & 3], 0, 0, 0);
  }
}

struct AttnKArgs {
  const bf16_t* qkv;
  const bf16_t* pk;
  const bf16_t* pv;
  bf16_t* out;
  float* opart;         // [nS][M][Hq][128]
  float* mlpart;        // [nS][M][Hq][2]
  int M, B, Hq, Hkv, P, S, ldp, ld, nQ, nS;   // ldp = rows allocated per KV head of the cache; S = suffix rows
  int own;                                     // 0: no own-block keys (queries that only read the cache)
  int split;                                   // cached rows per split: the P + S rows shared out evenly, whole tiles
  int qrows;                                   // query rows a workgroup owns: 128, or 96 / 64 / 32 when there are few workgroups (scheduling only)
};

// DUAL: the cache also holds rows of the tokens after the block (a.S > 0)
template <bool DUAL>
__device__ __forceinline__ void attn_prefix_body(const AttnKArgs& a, int bid) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const unsigned lds0 = (unsigned)(size_t)(lds_ptr_t)smem_raw;

  const int total = a.nQ * a.nS * a.Hq;
  const int L = xcd_contiguous(bid, total);
  const int qt = L % a.nQ;
  const int sp = (L / a.nQ) % a.nS;
  const int h = L / (a.nQ * a.nS);
  const int kvh = h / (a.Hq / a.Hkv);

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l32 = lane & 31, hh = lane >> 5;
  // query group of the wavefront pair, and this wavefront's role in it: the key half it takes (role 0 also takes the
  // own-block keys and finishes the pair's rows).  Role 0 sits on wavefronts 0, 2, 5, 7, one per SIMD when wavefronts go
  // round the four SIMDs in order: the four pairs' own-block phases and final merges then do not share SIMDs two by two.
  const int qw = wave >> 1, st = (wave ^ (wave >> 2)) & 1;
  const int m0 = qt * a.qrows;
  const int m_end = min(a.M, m0 + a.qrows);     // the workgroup's query rows are m0 .. m_end-1
  const int m0w = m0 + qw * 32;
  const int qrow = min(m0w + l32, a.M - 1);
  // A wavefront pair whose 32 query rows all lie beyond M (one or two states in a 128-row tile) takes part in the
  // transfers and barriers only: the pairs that do have rows then keep their SIMDs to themselves.
  const bool active = __builtin_amdgcn_readfirstlane(m0w) < m_end;

  WaveState w;
  w.m_run = -INFINITY;
  w.l_run = 0.f;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int v = 0; v < 16; ++v) w.o[n][v] = 0.f;

  // The cached keys form one axis of P + S rows: the prefix (cache rows 0 .. P-1), then the tokens after the
  // block (dual cache: cache rows P+B .. P+B+S-1).  Split `sp` owns a.split consecutive rows of that axis
  // and streams its prefix part, then its suffix part; [kbeg, kend) are cache rows of the part in progress.
  const int v0 = sp * a.split, v1 = min(a.P + a.S, v0 + a.split);
  int kbeg = min(v0, a.P);
  int kend = min(v1, a.P);
  int n_tiles = kend > kbeg ? (kend - kbeg + KTILE - 1) / KTILE : 0;
  const bf16_t* pk = a.pk + (size_t)kvh * a.ldp * HD;
  const bf16_t* pv = a.pv + (size_t)kvh * a.ldp * HD;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  // 16 bytes per lane, global (scalar base + 32-bit lane offset) -> LDS (M0 = destination of lane 0)
  auto dma16 = [&](const char* ubase, unsigned lane_off, unsigned dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds0 + dst), "v"(lane_off), "s"(ubase) : "memory");
  };
  // One wave-load brings four rows of 256 bytes: lane -> (row, LDS position) -> source chunk.  A 64-row tile takes two per
  // wavefront (rows 8*wave ..), 128 rows four (rows 16*wave ..).
  const int lrow = lane >> 4, lpos = lane & 15;
  const unsigned koff0 = (8 * wave_u + lrow) * (HD * 2) + k_pos(8 * wave_u + lrow, lpos) * 16;
  const unsigned koff1 = (8 * wave_u + 4 + lrow) * (HD * 2) + k_pos(8 * wave_u + 4 + lrow, lpos) * 16;
  const unsigned voff = (8 * wave_u + lrow) * (HD * 2) + v_pos(lrow, lpos) * 16;      // rows 4 further on: the same chunks
  auto issue_tile = [&](int t) {     // prefix tile t of this split into its ring stages
    const int row0 = kbeg + t * KTILE, nv = kend - row0;
    const char* kp = reinterpret_cast<const char*>(pk + (size_t)row0 * HD);
    const char* vp = reinterpret_cast<const char*>(pv + (size_t)row0 * HD);
    const unsigned dst = (t % NSTAGE) * STAGE_BYTES + wave_u * (8 * HD * 2);
    if (nv >= KTILE) {
      dma16(kp, koff0, dst);
      dma16(kp, koff1, dst + 4 * HD * 2);
      dma16(vp, voff, V_RING + dst);
      dma16(vp + 4 * HD * 2, voff, V_RING + dst + 4 * HD * 2);
    } else {                          // ragged last tile: rows beyond the end repeat the last one
      const unsigned r0 = 8 * wave_u + lrow, r1 = r0 + 4;
      const unsigned back0 = (r0 - min(r0, (unsigned)(nv - 1))) * (HD * 2), back1 = (r1 - min(r1, (unsigned)(nv - 1))) * (HD * 2);
      dma16(kp, koff0 - back0, dst);
      dma16(kp, koff1 - back1, dst + 4 * HD * 2);
      dma16(vp, voff - back0, V_RING + dst);
      dma16(vp, voff + 4 * HD * 2 - back1, V_RING + dst + 4 * HD * 2);
    }
  };
  // rows row0 .. row0+127 (clamped to M-1) of one head's columns of the fused activations: whole groups of 32 up to row_end
  // (a masked key of a group still multiplies its V row by 0)
  auto issue_rows128 = [&](unsigned dst, bool vswz, int col, int row0, int row_end) {
    if (16 * wave_u >= ((row_end - row0 + 31) & ~31)) return;
    const char* base = reinterpret_cast<const char*>(a.qkv + (size_t)row0 * a.ld + col);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = 16 * wave_u + 4 * q + lrow;
      const int chunk = vswz ? v_pos(row, lpos) : k_pos(row, lpos);
      dma16(base, (unsigned)min(row, a.M - 1 - row0) * (unsigned)(a.ld * 2) + chunk * 16, dst + (16 * wave_u + 4 * q) * (HD * 2));
    }
  };
  // own-block rows c0 .. c0+127 (K and V columns)
  const bool has_own = a.own && sp == a.nS - 1;
  // Groups of 32 keys are counted from the first row of the state that holds the first row of the 128-row tile (when B
  // divides 32 or 32 divides B that is a multiple of 32 for any tile); the workgroup starts with the group its rows need first.
  const int own0 = (((32 % a.B == 0 || a.B % 32 == 0) ? m0 : m0 & ~(QTILE - 1)) / a.B) * a.B;
  const int own_lo = own0 + (((m0 / a.B) * a.B - own0) & ~31);
  const int own_hi = min(a.M, ((m_end - 1) / a.B + 1) * a.B);
  auto issue_own = [&](int c0) {
    issue_rows128(OWN_K, false, (a.Hq + kvh) * HD, c0, own_hi);
    issue_rows128(OWN_V, true, (a.Hq + a.Hkv + kvh) * HD, c0, own_hi);
  };

  // ---- start every transfer known up front: Q, the first own-block rows, prefix tiles 0 and 1; all of them arrive as whole
  // 256-byte rows.  Q and the own rows are waited for, the tiles stay in flight.
  issue_rows128(Q_ROWS, false, h * HD, m0, m_end);
  if (has_own) issue_own(own_lo);
  if (n_tiles > 0) issue_tile(0);
  if (n_tiles > 1) { issue_tile(1); wait_vmcnt<2 * DMA_PER_TILE>(); }
  else if (n_tiles == 1) wait_vmcnt<DMA_PER_TILE>();
  else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();

  // ---- Q: fragments of the wavefront pair's rows
  {
    const KAddr qa = k_addr(lds0 + Q_ROWS, qw * 32, lane);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) w.qf[kk] = k_frag<0>(qa, kk);
  }

  // ---- own-block keys: the block diagonal, handled by the last split.  They always go to the role-0 wavefront
  // of the pair, 32 keys at a time in row order.
  if (has_own) {
    // rows of the states this wave's queries belong to
    const int w_lo = (min(m0w, a.M - 1) / a.B) * a.B;
    const int w_hi = (min(m0w + 31, a.M - 1) / a.B + 1) * a.B;
    const int q_lo = (qrow / a.B) * a.B;    // this lane's state: rows [q_lo, q_hi)
    const int q_hi = min(q_lo + a.B, a.M);
    for (int c0 = own_lo; c0 < own_hi; c0 += 128) {
      if (c0 != own_lo) {      // more than 128 own rows: next chunk
        __syncthreads();
        issue_own(c0);
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
      }
      if (st == 0 && active) {
#pragma nounroll
        for (int sub = 0; sub < 4; ++sub) {
          const int k_lo = c0 + sub * 32;
          if (k_lo < w_hi && k_lo + 32 > w_lo && k_lo < own_hi) {   // wave-uniform: this group holds keys of my states
            f32x16 sc;
            scores<0>(w, sc, k_addr(lds0 + OWN_K, sub * 32, lane));
            finish_masked(w, sc, v_addr(lds0 + OWN_V, sub * 32, lane), lane,
                          [k_lo, q_lo, q_hi](int key) { return k_lo + key >= q_lo && k_lo + key < q_hi; });
          }
        }
      }
    }
  }
  __syncthreads();   // Q and own-block rows are consumed: stages 2 and 3 are free

  // ---- cached keys of this split: LDS-DMA rings, up to NSTAGE-1 tiles ahead --------------------------
#pragma nounroll
  for (int part = 0; part < (DUAL ? 2 : 1); ++part) {
  if (part == 1) {
    kbeg = max(v0, a.P) + a.B;
    kend = max(v1, a.P) + a.B;
    n_tiles = kend > kbeg ? (kend - kbeg + KTILE - 1) / KTILE : 0;
    if (n_tiles > 0) issue_tile(0);      // the ring is drained: every stage is free
    if (n_tiles > 1) issue_tile(1);
  }
  if (n_tiles == 0) continue;
  if (2 < n_tiles) issue_tile(2);
  // full tiles run through the software pipeline (scores of tile t+1 under the softmax of tile t); a ragged
  // last tile, whose scores come out of it too, takes the masked path afterwards
  const bool ragged = ((kend - kbeg) % KTILE) != 0;
  const int n_pipe = ragged ? n_tiles - 1 : n_tiles;
  KAddr ka = k_addr(lds0, st * 32, lane);
  VAddr va = v_addr(lds0 + V_RING, st * 32, lane);
  // tile 0 has landed; tiles 1 .. min(2, n_tiles-1) may still be in flight
  if (n_tiles >= 3) wait_vmcnt<2 * DMA_PER_TILE>(); else if (n_tiles == 2) wait_vmcnt<DMA_PER_TILE>(); else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  f32x16 sa, sb;
  if (active) scores<0>(w, sa, ka);
  // step t: tile t+1 has landed (tile t+2 may be in flight) and every wavefront is done with step t-1,
  // i.e. with K of tile t and V of tile t-1, whose stage the next prefetch overwrites
  auto sync_and_prefetch = [&](int t) {
    if (t + 2 < n_tiles) wait_vmcnt<DMA_PER_TILE>(); else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    if (t + NSTAGE - 1 < n_tiles) issue_tile(t + NSTAGE - 1);
  };
  // Two steps per trip: the score registers swap roles and the addresses move on by two stages, alternately up and down
  // (K of tile t+1 sits one stage ahead of V of tile t, so its addresses move between the steps).  The step of the last
  // tile also takes scores of whatever the next stage holds; nothing reads them.
  unsigned hop = 2 * STAGE_BYTES;
  int t = 0;
  for (; t + 1 < n_pipe; t += 2) {
    sync_and_prefetch(t);
    if (active) pipe_step<STAGE_BYTES, 0>(w, sa, sb, ka, va);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) ka.a[kk] += hop;
    sync_and_prefetch(t + 1);
    if (active) pipe_step<0, STAGE_BYTES>(w, sb, sa, ka, va);
#pragma unroll
    for (int n = 0; n < 4; ++n) va.a[n] += hop;
    hop = 0u - hop;
  }
  if (t < n_pipe) {
    sync_and_prefetch(t);
    if (active) pipe_step<STAGE_BYTES, 0>(w, sa, sb, ka, va);
    sa = sb;
  }
  if (ragged && active) {
    const int nvalid = kend - (kbeg + n_pipe * KTILE) - st * 32;
    finish_masked(w, sa, v_addr(lds0 + V_RING + (n_pipe % NSTAGE) * STAGE_BYTES, st * 32, lane), lane,
                  [nvalid](int key) { return key < nvalid; });
  }
  __syncthreads();   // all tiles consumed, no DMA in flight: the ring can be reused
  }
  // ---- merge the two key halves of each wavefront pair through LDS ------------------------------
  {
    float* xb = reinterpret_cast<float*>(smem_raw) + (size_t)qw * 66 * 64;   // [66][64 lanes] per pair
    if (st == 1) {
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) xb[(n * 16 + v) * 64 + lane] = w.o[n][v];
      xb[64 * 64 + lane] = w.m_run;
      xb[65 * 64 + lane] = w.l_run;
    }
    __syncthreads();
    if (st == 1) return;
    const float m1 = xb[64 * 64 + lane], l1 = xb[65 * 64 + lane];
    const float mm = fmaxf(w.m_run, m1);
    const float a0 = (w.m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(w.m_run - mm);
    const float a1 = (m1 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m1 - mm);
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int v = 0; v < 16; ++v) w.o[n][v] = w.o[n][v] * a0 + xb[(n * 16 + v) * 64 + lane] * a1;
    w.l_run = w.l_run * a0 + l1 * a1;
    w.m_run = mm;
  }

  // ---- write ----------------------------------------------------------------------------------
  const float l_tot = w.l_run + __shfl_xor(w.l_run, 32, 64);
  if (m0w + l32 >= m_end) return;
  if (a.nS == 1) {
    const float inv = 1.0f / l_tot;
    bf16_t* op = a.out + (size_t)qrow * (a.Hq * HD) + h * HD + 4 * hh;
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = static_cast<bf16_t>(w.o[n][g4 * 4 + e] * inv);
        *reinterpret_cast<bf16x4*>(op + n * 32 + g4 * 8) = t;
      }
  } else {
    const size_t rowh = ((size_t)sp * a.M + qrow) * a.Hq + h;
    float* op = a.opart + rowh * HD + 4 * hh;
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        f32x4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = w.o[n][g4 * 4 + e];
        *reinterpret_cast<f32x4*>(op + n * 32 + g4 * 8) = t;
      }
    if (hh == 0) {
      a.mlpart[rowh * 2] = w.m_run;
      a.mlpart[rowh * 2 + 1] = l_tot;
    }
  }
}

template <bool DUAL>
__global__ __launch_bounds__(NT) void attn_prefix_mfma_kernel(AttnKArgs a) {
  attn_prefix_body<DUAL>(a, (int)blockIdx.x);
}

// Two independent attention problems in one launch (the G states and, beside them, the rows that ride along with a
// step: the recomputed suffix, or the block being committed): the first n_a workgroups take `a`, the rest `b`.
// Each part alone would leave most CUs idle when there are few states.
__global__ __launch_bounds__(NT) void attn_prefix_mfma_pair_kernel(AttnKArgs a, AttnKArgs b, int n_a) {
  if ((int)blockIdx.x < n_a) attn_prefix_body<true>(a, (int)blockIdx.x);
  else attn_prefix_body<true>(b, (int)blockIdx.x - n_a);
}

// merge the prefix splits of each (row, head): weights 2^(m_s - max m).  32 lanes per (row, head), four head
// dimensions per lane, eight (row, head) pairs per workgroup.
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ opart,
                                                           const float* __restrict__ mlpart, bf16_t* __restrict__ out,
                                                           int M, int Hq, int nS) {
  const size_t n_rowh = (size_t)M * Hq;
  const size_t rowh = (size_t)blockIdx.x * 8 + (threadIdx.x >> 5);   // row * Hq + head
  if (rowh >= n_rowh) return;
  const int t = (threadIdx.x & 31) * 4;
  float mx = -INFINITY;
  for (int s = 0; s < nS; ++s) mx = fmaxf(mx, mlpart[((size_t)s * n_rowh + rowh) * 2]);
  f32x4 num = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f;
  for (int s = 0; s < nS; ++s) {
    const size_t i = (size_t)s * n_rowh + rowh;
    const float ms = mlpart[i * 2];
    const float wgt = (ms == -INFINITY) ? 0.f : exp2f(ms - mx);
    den += wgt * mlpart[i * 2 + 1];
    const f32x4 o = *reinterpret_cast<const f32x4*>(opart + i * HD + t);
#pragma unroll
    for (int e = 0; e < 4; ++e) num[e] += wgt * o[e];
  }
  bf16x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = static_cast<bf16_t>(num[e] / den);
  *reinterpret_cast<bf16x4*>(out + rowh * HD + t) = r;
}

inline int n_splits(int P) { return P > 0 ? cdiv(P, SPLIT_KEYS) : 1; }

}  // namespace

// split partials; P = cached keys, prefix and suffix together
size_t mfma_attn_partial_bytes(int G, int B, int Hq, int hd, int P) {
  const size_t M = (size_t)G * B;
  size_t bytes = 0;
  const int nS = n_splits(P);
  if (nS > 1) {
    bytes += align_up(sizeof(float) * nS * M * Hq * hd, 256);
    bytes += align_up(sizeof(float) * nS * M * Hq * 2, 256);
  }
  return bytes;
}

namespace {

// kernel arguments of one attention problem
AttnKArgs prepare_attn(const AttnArgs& a) {
  const int M = a.G * a.B;
  const int nS = n_splits(a.P + a.S);
  unsigned char* ws = reinterpret_cast<unsigned char*>(a.partial);
  float* opart = reinterpret_cast<float*>(ws);
  ws += align_up(sizeof(float) * (size_t)nS * M * a.Hq * HD, 256);
  float* mlpart = reinterpret_cast<float*>(ws);

  AttnKArgs k;
  k.qkv = (const bf16_t*)a.qkv;
  k.pk = (const bf16_t*)a.prefix_k;
  k.pv = (const bf16_t*)a.prefix_v;
  k.out = (bf16_t*)a.out;
  k.opart = opart;
  k.mlpart = mlpart;
  k.M = M; k.B = a.B; k.Hq = a.Hq; k.Hkv = a.Hkv; k.P = a.P; k.S = a.S; k.ldp = a.ldp ? a.ldp : a.P;
  k.own = a.own;
  k.ld = (a.Hq + 2 * a.Hkv) * HD;
  // With few workgroups (one to eight states) a workgroup takes 64 or 32 query rows instead of 128, so that more CUs
  // stream the keys; the wavefront pairs without rows only move data.  A row's arithmetic is the same: the groups of own-block
  // keys are those of the 128-row tile.
  k.qrows = QTILE;
  const int wgs = cdiv(M, QTILE) * nS * a.Hq;
  if (wgs <= 64) k.qrows = 32;
  else if (wgs <= 128) k.qrows = 64;
  // between half and the whole chip (28 heads x 6 tiles of 128 rows = 168 workgroups): 96 rows, three of the four
  // wavefront pairs at work, if that brings more workgroups and still one round of them (28 x 8 = 224)
  // (96 rows do not lie inside one tile of 128: for blocks whose groups of own keys start anywhere 128 rows stay)
  else if (wgs < 256 && cdiv(M, 96) > cdiv(M, QTILE) && cdiv(M, 96) * nS * a.Hq <= 256 &&
           (!a.own || 32 % a.B == 0 || a.B % 32 == 0)) k.qrows = 96;
  k.nQ = cdiv(M, k.qrows);
  k.nS = nS;
  k.split = (int)align_up(cdiv(a.P + a.S, nS), KTILE);      // at most SPLIT_KEYS; a function of P + S only
  return k;
}

hipError_t attn_lds_limits() {
  static std::atomic<unsigned long long> lds_ok[3];
  hipError_t e = allow_dynamic_lds((const void*)attn_prefix_mfma_kernel<false>, (int)kAttnSmem, lds_ok[0]);
  if (e != hipSuccess) return e;
  e = allow_dynamic_lds((const void*)attn_prefix_mfma_kernel<true>, (int)kAttnSmem, lds_ok[1]);
  if (e != hipSuccess) return e;
  return allow_dynamic_lds((const void*)attn_prefix_mfma_pair_kernel, (int)kAttnSmem, lds_ok[2]);
}

}  // namespace

hipError_t launch_attn_mfma(const AttnArgs& a, hipStream_t st) {
  const hipError_t e = attn_lds_limits();
  if (e != hipSuccess) return e;
  const AttnKArgs k = prepare_attn(a);
  const int grid = k.nQ * k.nS * a.Hq;
  if (a.S > 0) attn_prefix_mfma_kernel<true><<<grid, NT, kAttnSmem, st>>>(k);
  else attn_prefix_mfma_kernel<false><<<grid, NT, kAttnSmem, st>>>(k);
  if (k.nS > 1) attn_combine_kernel<<<cdiv(k.M * a.Hq, 8), 256, 0, st>>>(k.opart, k.mlpart, k.out, k.M, a.Hq, k.nS);
  return hipGetLastError();
}

// two independent problems (different query rows, outputs and scratch; they may read the same cache) in one launch
hipError_t launch_attn_mfma_pair(const AttnArgs& a, const AttnArgs& b, hipStream_t st) {
  const hipError_t e = attn_lds_limits();
  if (e != hipSuccess) return e;
  const AttnKArgs ka = prepare_attn(a), kb = prepare_attn(b);
  const int n_a = ka.nQ * ka.nS * a.Hq, n_b = kb.nQ * kb.nS * b.Hq;
  attn_prefix_mfma_pair_kernel<<<n_a + n_b, NT, kAttnSmem, st>>>(ka, kb, n_a);
  if (ka.nS > 1) attn_combine_kernel<<<cdiv(ka.M * a.Hq, 8), 256, 0, st>>>(ka.opart, ka.mlpart, ka.out, ka.M, a.Hq, ka.nS);
  if (kb.nS > 1) attn_combine_kernel<<<cdiv(kb.M * b.Hq, 8), 256, 0, st>>>(kb.opart, kb.mlpart, kb.out, kb.M, b.Hq, kb.nS);
  return hipGetLastError();
}

}  // namespace spiffy
