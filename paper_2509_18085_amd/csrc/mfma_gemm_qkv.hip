// Tile shapes of the rotary epilogue (mfma_gemm_kernel.h).
#include "mfma_gemm_kernel.h"

namespace spiffy {

hipError_t launch_gemm_qkv(const GemmArgs& a, TileShape t, hipStream_t st) { return launch_shape<EPI_QKV>(a, t, st); }

}  // namespace spiffy
