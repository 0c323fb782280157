// gate/up projection with the SwiGLU epilogue, 128-row n-blocks (tile counts no multiple of three)
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_swiglu_wn4(const GemmArgs& a) { return launch_shape<4, EPI_SWIGLU>(a); }
