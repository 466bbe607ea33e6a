#pragma once
// bf16 MFMA GEMM for gfx950:  D[i,j] = sum_k X[i,k] * Y[j,k]  (both operands K-contiguous), fp32
// accumulation with v_mfma_f32_32x32x16_bf16.
//
// Shape of the kernel (what measurements on MI355X pushed it to):
//   * one workgroup per CU: 256 x BN output tile (BN = 256, 192 or 128), 4 wavefronts in a 2x2 grid, each
//     wavefront owns 128 x BN/2 (accumulators in AGPRs; 192 to 384 rows where they fill the rounds better).  The L2 delivers about 32 B/clk to a CU, so
//     a tile needs >= 64..128 flop per loaded byte; 128x128 tiles are bound by that, 256x192 is not.
//     With few rows (one to eight states) the projections only stream weights: the same kernel with
//     128- or 64-row tiles does half or a quarter of the matrix work per tile and covers more CUs; the
//     narrow split-K projections of one or two states take 32-column tiles with one wavefront along a
//     32-wide side (64 x 32: two wavefronts, 32 x 32: one), so 256 workgroups stream instead of 128;
//     the gate/up projection of up to 128 rows takes 96-column tiles (256 workgroups instead of 192):
//     a 1 x 4 wavefront grid, three wavefronts own a 32-column block each, the fourth only loads.
//   * K advances in steps of 64 so every row segment is one full 128-byte line; operands go
//     global -> LDS directly (LDS-DMA loads, no register staging), rows XOR-swizzled so the
//     16-byte fragment reads are conflict-free.
//   * separate LDS rings for the two operands: the activation operand (mostly L2 hits) gets 2 stages,
//     the weight operand (streamed from HBM) SD = 3-4 stages, 128-144 KB in all.
//   * one barrier per K-tile; the loads of later tiles and the LDS fragment reads of the next
//     16-wide K step are threaded between the MFMAs of the current step, fragments double-buffered
//     in registers, partial s_waitcnt vmcnt so younger loads stay in flight across the barrier.
//   * workgroup ids are remapped so that the workgroups sharing a weight tile sit on one XCD.
//
// Epilogues:
//   EPI_STORE    C = X W^T
//   EPI_QKV      C = X [Wq | Wk | Wv]^T (+ biases), heads of 128 columns, with the rotary embedding on the q and k
//                columns: a 32-column MFMA tile holds 16 columns c and the 16 columns c + 64 of a head, partner
//                values are in one lane; k and v rows that extend the cache are stored there too
//   EPI_RESID    C = R + X W^T
//   EPI_SWIGLU   C = silu(X Wg^T) * (X Wu^T); gate and up rows are interleaved 16/16 inside every
//                32-column MFMA tile, partner values are in one lane
//   EPI_PARTIAL  fp32 partial sums of one K slice (split-K for narrow N; reduced by a second kernel
//                in a fixed order, the slice count depends on (N, K) only)
//   EPI_LMHEAD   rows i = vocabulary entries, columns j = tokens: each lane owns token columns and
//                reduces its logits to (top, lowest index, runner-up, sum exp) in registers; logits
//                are never stored (Alg. 1 steps 1-2 fused into the GEMM)
//
// The accumulation order along K of every output element is fixed by (N, K) alone, so a row's result
// does not depend on how many other states are verified with it.
#include <type_traits>

#include "kernels.h"

namespace spiffy {

namespace {

constexpr int BM = 256, BKK = 64;

typedef __attribute__((address_space(3))) void* lds_ptr_t;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {   // vmcnt <= N; lgkmcnt / expcnt untouched
  __builtin_amdgcn_s_waitcnt((N & 0xF) | (7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// 64-row tiles, and 128-row tiles up to 128 columns wide, are weight-streaming shapes: both operand rings SD deep
constexpr bool uniform_rings(int epi, int bn, int bmt) { return epi != EPI_LMHEAD && (bmt <= 64 || (bmt == 128 && bn <= 128)); }
// stages of the shallow operand's ring = how many K-tiles ahead it is loaded; SA = 0 picks the default of the shape
constexpr int shallow_stages(int epi, int bn, int bmt, int sd, int sa) { return sa ? sa : (uniform_rings(epi, bn, bmt) ? sd : 2); }
// wavefronts of a workgroup: a 2 x 2 grid over the tile; a 32-row or 32-column tile has one wavefront along that side.
// A 96-column tile (three 32-column blocks: what gives 256 workgroups when 128 columns give 192) has a 1 x 4 grid whose
// first three wavefronts own one block each; the fourth only takes its share of the loads.
// The LM head's 128-row tile has a 1 x 4 grid too: a wavefront's 128 vocabulary rows are one part of the summaries.
constexpr bool one_by_four(int epi, int bmt, int bn) { return bn == 96 || (epi == EPI_LMHEAD && bmt == 128); }
constexpr int waves_m(int epi, int bmt, int bn) { return one_by_four(epi, bmt, bn) ? 1 : (bmt >= 64 ? 2 : 1); }
constexpr int waves_n(int epi, int bmt, int bn) { return one_by_four(epi, bmt, bn) ? 4 : (bn >= 64 ? 2 : 1); }
constexpr int wave_cols(int epi, int bmt, int bn) { return bn == 96 ? 32 : bn / waves_n(epi, bmt, bn); }

// the wavefront id is uniform: keep it (and all LDS destination arithmetic) in scalar registers
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// The lane id, counted at every call: the head's epilogue does not keep the K loop's copy (or threadIdx) alive over all its
// shapes, of which one fills the 512 registers: a kernel with scratch memory starts some 3 us later.
__device__ __forceinline__ int lane_id() {
  unsigned all = ~0u;
  asm volatile("" : "+s"(all));
  return __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

// One output tile: the kernel of the projections, and a function for the head, which picks one of several shapes on the device.
// The body is a file of its own, included in both: as a function called by both kernels the compiler kept the arguments in other
// registers (QKV 6% longer, gate/up of 128 rows 47.1 -> 49.9 us).
template <int EPI, int BN, int SD, int BMT = 256, int SA = 0>
__global__ __launch_bounds__(256) void gemm_bf16_mfma_kernel(GemmArgs a, int tiles_i, int tiles_j) {
  const int wave = wave_id();
#include "mfma_gemm_body.h"
}

template <int EPI, int BN, int SD, int BMT, int SA>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, int tiles_i, int tiles_j, int wave) {
#include "mfma_gemm_body.h"
}

template <int EPI, int BN, int SD, int BMT, int SA>
constexpr size_t smem_bytes() {
  constexpr int SH = shallow_stages(EPI, BN, BMT, SD, SA);
  return sizeof(bf16_t) * (size_t)(EPI == EPI_LMHEAD ? SD * BMT + SH * BN : SH * BMT + SD * BN) * BKK;
}

template <int EPI, int BN, int SD, int BMT = 256, int SA = 0>
hipError_t launch_t(const GemmArgs& a, int tiles_i, int tiles_j, hipStream_t st) {
  static_assert(smem_bytes<EPI, BN, SD, BMT, SA>() <= 160 * 1024, "a workgroup has 160 KB of LDS");
  static std::atomic<unsigned long long> lds_ok{0};
  const hipError_t e = allow_dynamic_lds((const void*)gemm_bf16_mfma_kernel<EPI, BN, SD, BMT, SA>,
                                         (int)smem_bytes<EPI, BN, SD, BMT, SA>(), lds_ok);
  if (e != hipSuccess) return e;
  gemm_bf16_mfma_kernel<EPI, BN, SD, BMT, SA><<<tiles_i * tiles_j * a.ksplit, 64 * waves_m(EPI, BMT, BN) * waves_n(EPI, BMT, BN), smem_bytes<EPI, BN, SD, BMT, SA>(), st>>>(a, tiles_i, tiles_j);
  return hipGetLastError();
}

// The tile shapes of each epilogue: what launch_shape instantiates and the rules may pick.
constexpr bool has_shape(int epi, int bm, int bn) {
  switch (bm * 1000 + bn) {
    case 256128: case 256064: case 128128: case 64128: case 64064: return true;
    case 256192: case 128192: case 128096: case 64096: return epi != EPI_PARTIAL;      // the split-K projections are narrow
    case 64032: case 32032: return epi == EPI_PARTIAL;
    case 192128: case 128064: case 320128: return epi != EPI_STORE;                    // heights in between: a layer's own launches
    case 192192: case 256256: return epi == EPI_QKV || epi == EPI_SWIGLU;
    case 320192: case 384128: return epi == EPI_SWIGLU;
    default: return false;
  }
}

template <int EPI, int BN, int SD, int BMT, int SA = 0>
bool launch_if(const GemmArgs& a, TileShape t, hipStream_t st, hipError_t& e) {
  if constexpr (has_shape(EPI, BMT, BN)) {
    if (t.bm == BMT && t.bn == BN) {
      e = launch_t<EPI, BN, SD, BMT, SA>(a, cdiv(a.M, BMT), a.N / (BN / (EPI == EPI_SWIGLU ? 2 : 1)), st);
      return true;
    }
  }
  return false;
}

// One launch in tiles of shape t over all of a.N columns (SWIGLU: features).  The few-row shapes have weight rings as deep as
// the LDS allows: bytes in flight are what sets the streaming rate.
template <int EPI>
hipError_t launch_shape(const GemmArgs& a, TileShape t, hipStream_t st) {
  constexpr bool SWIGLU = EPI == EPI_SWIGLU;
  hipError_t e = hipErrorInvalidValue;
  // 256 x 128: room for a third activation stage beside four weight stages (160 KB); in interleaved A/B runs 2-5%
  // faster than two stages on every projection that takes this tile (down projection 95.9 -> 91.4 us at 1024 rows)
  (void)(launch_if<EPI, 128, 4, 256, 3>(a, t, st, e) || launch_if<EPI, 64, 4, 256>(a, t, st, e) ||
         launch_if<EPI, 128, 4, 128>(a, t, st, e) || launch_if<EPI, 128, 6, 64>(a, t, st, e) ||
         launch_if<EPI, 64, 8, 64>(a, t, st, e) || launch_if<EPI, 192, 3, 256>(a, t, st, e) ||
         launch_if<EPI, 192, 4, 128>(a, t, st, e) || launch_if<EPI, 96, SWIGLU ? 5 : 4, 128>(a, t, st, e) ||
         launch_if<EPI, 96, SWIGLU ? 7 : 6, 64>(a, t, st, e) || launch_if<EPI, 32, 10, 64>(a, t, st, e) ||
         launch_if<EPI, 32, 9, 32>(a, t, st, e) || launch_if<EPI, 128, 4, 192, 4>(a, t, st, e) ||
         launch_if<EPI, 64, 6, 128>(a, t, st, e) || launch_if<EPI, 128, 4, 320, 2>(a, t, st, e) ||
         launch_if<EPI, 192, 3, 192, 3>(a, t, st, e) || launch_if<EPI, 256, 3, 256>(a, t, st, e) ||
         launch_if<EPI, 192, 3, 320>(a, t, st, e) || launch_if<EPI, 128, 4, 384, 2>(a, t, st, e));
  return e;
}

}  // namespace

}  // namespace spiffy
