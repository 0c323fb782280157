// fp32 partial sums, 64-row n-blocks (the attention output projection)
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_f32_wn2(const GemmArgs& a) { return launch_shape<2, EPI_F32>(a); }
