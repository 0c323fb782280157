// fp32 partial sums, 128-row n-blocks (the down projection): 24 chunks per k-slice at d_ffn 12288
// (one instantiation unit of the MFMA GEMM template; see kernels_mfma.hip for the design)
#include "gemm_mfma.h"

bool gemm_f32_wn4(const GemmArgs& a) { return launch_shape<4, 2, EPI_F32, 24>(a); }
