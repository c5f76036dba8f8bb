// Body of product_dispatch<MODE, BT>: maps the run-time launch shape onto the instantiations of product_kernel.
// Included by the bb_product_inst_*.hip sources, each of which instantiates it for one MODE and one weight layout.
#pragma once
#include "bb_launch.h"
#include "bb_product.h"

namespace bb {

template <int MODE, bool BT>
void product_dispatch(int bm, int bn, int parts, dim3 grid, hipStream_t st, const GemmArgs& a) {
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(PRODUCT_THREADS), 0, st, a); };
    auto by_tile = [&](auto RAGGEDc) {
        constexpr bool R = decltype(RAGGEDc)::value;
        if constexpr (MODE == MODE_PLAIN) {
            if (parts == PARTS_FOLD) return go(product_kernel<MODE, 128, 128, PARTS_FOLD, BT, R>);
            if (parts == PARTS_APART && bn == 128) return go(product_kernel<MODE, 128, 128, PARTS_APART, BT, R>);
            if (parts == PARTS_APART)
                return bm == 128 ? go(product_kernel<MODE, 128, 256, PARTS_APART, BT, R>) : go(product_kernel<MODE, 256, 256, PARTS_APART, BT, R>);
            if (bn == 128) return go(product_kernel<MODE, 128, 128, PARTS_ONE, BT, R>);
        }
        if (bm == 128) go(product_kernel<MODE, 128, 256, PARTS_ONE, BT, R>); else go(product_kernel<MODE, 256, 256, PARTS_ONE, BT, R>);
    };
    if (a.K % GEMM_BK) by_tile(std::true_type()); else by_tile(std::false_type());
}

}  // namespace bb
