// fp32 partial sums, 96-row n-blocks (the QKV projection)
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_f32_wn3(const GemmArgs& a) { return launch_shape<3, EPI_F32>(a); }
