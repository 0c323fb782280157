// many-row GEMM, EPI_F32 epilogue (one instantiation unit of gemm_rows.h)
#include "gemm_rows.h"

bool gemm_rows_f32(const GemmArgs& a, int mt) {
    switch (mt) {
        case 3: return launch_rows<3, EPI_F32, 4, 4>(a);
        case 4: return launch_rows<4, EPI_F32, 4, 4>(a);
        case 5: return launch_rows<5, EPI_F32, 2, 4>(a);
    }
    return false;
}
