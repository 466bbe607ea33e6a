// Tile shapes of the gate/up epilogue (mfma_gemm_kernel.h).
#include "mfma_gemm_kernel.h"

namespace spiffy {

hipError_t launch_gemm_swiglu(const GemmArgs& a, TileShape t, hipStream_t st) { return launch_shape<EPI_SWIGLU>(a, t, st); }

}  // namespace spiffy
