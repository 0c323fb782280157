// many-row GEMM, EPI_LMHEAD epilogue (one instantiation unit of gemm_rows.h)
#include "gemm_rows.h"

bool gemm_rows_lmhead(const GemmArgs& a, int mt) {
    switch (mt) {
        case 3: return launch_rows<3, EPI_LMHEAD, 4, 4>(a);
        case 4: return launch_rows<4, EPI_LMHEAD, 4, 4>(a);
        case 5: return launch_rows<5, EPI_LMHEAD, 2, 4>(a);
    }
    return false;
}
