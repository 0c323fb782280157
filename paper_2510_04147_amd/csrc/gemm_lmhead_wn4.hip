// LM head with the per-tile (max, arg-max, sum-exp) reduction, 128-row n-blocks
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_lmhead_wn4(const GemmArgs& a) { return launch_shape<4, EPI_LMHEAD>(a); }
