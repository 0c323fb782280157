// fp32 partial sums, 128-row n-blocks (the down projection)
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_f32_wn4(const GemmArgs& a) { return launch_shape<4, EPI_F32>(a); }
