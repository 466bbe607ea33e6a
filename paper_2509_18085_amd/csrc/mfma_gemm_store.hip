// Tile shapes of the plain store epilogue (mfma_gemm_kernel.h).
#include "mfma_gemm_kernel.h"

namespace spiffy {

hipError_t launch_gemm_store(const GemmArgs& a, TileShape t, hipStream_t st) { return launch_shape<EPI_STORE>(a, t, st); }

}  // namespace spiffy
