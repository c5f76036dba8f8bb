// few_rows_kernel and few_reduce_kernel instantiations and their launches
#include "bb_few.h"
#include "bb_launch.h"

namespace bb {

void few_rows_launch(int mt, bool bt, int grid, hipStream_t st, const FewArgs& a) {
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(FEW_THREADS), 0, st, a); };
    switch (mt) {
        case 1: bt ? go(few_rows_kernel<1, true>) : go(few_rows_kernel<1, false>); break;
        case 2: bt ? go(few_rows_kernel<2, true>) : go(few_rows_kernel<2, false>); break;
        case 3: bt ? go(few_rows_kernel<3, true>) : go(few_rows_kernel<3, false>); break;
        default: bt ? go(few_rows_kernel<4, true>) : go(few_rows_kernel<4, false>); break;
    }
}

void few_reduce_launch(int mode, hipStream_t st, const FewArgs& a, const float* rowstat, u16* C, int M,
                       const u16* res) {
    const dim3 grid(a.tiles_n, (M + FEW_RROWS - 1) / FEW_RROWS), block(32 * FEW_RROWS);
    if (mode == MODE_GATEUP_PRE)
        hipLaunchKernelGGL(few_reduce_kernel<MODE_GATEUP_PRE>, grid, block, 0, st, a, rowstat, C, M, res);
    else if (mode == MODE_LN_PRE)
        hipLaunchKernelGGL(few_reduce_kernel<MODE_LN_PRE>, grid, block, 0, st, a, rowstat, C, M, res);
    else
        hipLaunchKernelGGL(few_reduce_kernel<MODE_PLAIN>, grid, block, 0, st, a, rowstat, C, M, res);
}

}  // namespace bb
