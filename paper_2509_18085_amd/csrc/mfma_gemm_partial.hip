// Tile shapes of the split-K epilogue (mfma_gemm_kernel.h).
#include "mfma_gemm_kernel.h"

namespace spiffy {

hipError_t launch_gemm_partial(const GemmArgs& a, TileShape t, hipStream_t st) { return launch_shape<EPI_PARTIAL>(a, t, st); }

}  // namespace spiffy
