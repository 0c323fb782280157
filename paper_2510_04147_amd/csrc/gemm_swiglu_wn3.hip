// gate/up projection with the SwiGLU epilogue, 96-row n-blocks
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_swiglu_wn3(const GemmArgs& a) { return launch_shape<3, EPI_SWIGLU>(a); }
