// many-row GEMM, EPI_F32 epilogue (one instantiation unit of gemm_rows.h)
#include "gemm_rows.h"

bool gemm_rows_f32(const GemmArgs& a, int tile) { return launch_tile<EPI_F32>(a, tile); }
