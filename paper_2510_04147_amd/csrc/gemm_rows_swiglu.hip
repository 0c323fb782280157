// many-row GEMM, EPI_SWIGLU epilogue (one instantiation unit of gemm_rows.h)
#include "gemm_rows.h"

bool gemm_rows_swiglu(const GemmArgs& a, int tile) { return launch_tile<EPI_SWIGLU>(a, tile); }
