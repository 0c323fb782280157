// many-row GEMM, EPI_LMHEAD epilogue (one instantiation unit of gemm_rows.h)
#include "gemm_rows.h"

bool gemm_rows_lmhead(const GemmArgs& a, int tile) { return launch_tile<EPI_LMHEAD>(a, tile); }
