// Bodies of the attention launch functions: map the run-time launch shape onto
// the instantiations of the attention kernels.  Included by bb_attn_inst_*.hip,
// one source per pair of head dimensions.
#pragma once
#include <type_traits>

#include "bb_attn.h"
#include "bb_launch.h"

namespace bb {

// tail: iterations left after the two-per-trip main loop (1..4); nw: wavefronts per workgroup (4 or 8);
// ksplit > 1: keys split over ksplit workgroups per (problem, query block), then the combine kernel; flat (four wavefronts, d =
// dv = 128, tail 3 or 4): the FLAT kernels
template <int DK, int DV>
void attn_tiled_launch(int tail, int nw, int ksplit, bool flat, dim3 grid, dim3 block, hipStream_t st, const AttnArgs& a) {
    using T = std::true_type;
    using F_ = std::false_type;
    auto go = [&](auto NWC, auto KSPLITC, auto FLATC) {
        constexpr int NW = decltype(NWC)::value;
        constexpr bool KS = decltype(KSPLITC)::value, FL = decltype(FLATC)::value;
        if (!FL && tail == 1) hipLaunchKernelGGL((attention_kernel<DK, DV, 1, NW, KS>), grid, block, 0, st, a);
        else if (!FL && tail == 2) hipLaunchKernelGGL((attention_kernel<DK, DV, 2, NW, KS>), grid, block, 0, st, a);
        else if (tail == 3) hipLaunchKernelGGL((attention_kernel<DK, DV, 3, NW, KS, FL>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((attention_kernel<DK, DV, 4, NW, KS, FL>), grid, block, 0, st, a);
    };
    auto four = [&](auto KSPLITC) {
        using W4 = std::integral_constant<int, 4>;
        if constexpr (DK == 128 && DV == 128) {
            if (flat) return go(W4(), KSPLITC, T());
        }
        go(W4(), KSPLITC, F_());
    };
    if (ksplit > 1) {
        four(T());
        hipLaunchKernelGGL((attention_combine_kernel<DV>), dim3((unsigned)((size_t)a.B * a.M)), dim3(64), 0, st,
                           (const float*)a.part, (const float*)a.ml, a.O, ksplit, a.c);
    } else if (nw == 8) {
        go(std::integral_constant<int, 8>(), F_(), F_());
    } else {
        four(F_());
    }
}

template <int DK, int DV>
void attn_decode_launch(dim3 grid, hipStream_t st, const AttnArgs& a) {
    hipLaunchKernelGGL((attention_decode_kernel<DK, DV>), grid, dim3(256), 0, st, a);
}

template <int DK, int DV>
void attn_group_launch(int mt, dim3 grid, hipStream_t st, const AttnArgs& a) {
    if (mt == 1) hipLaunchKernelGGL((attention_group_kernel<DK, DV, 1>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((attention_group_kernel<DK, DV, 2>), grid, dim3(256), 0, st, a);
    if (a.nsplit > 1)
        hipLaunchKernelGGL((attention_combine_kernel<DV>), dim3((unsigned)((size_t)a.B * a.M)), dim3(64), 0, st,
                           (const float*)a.part, (const float*)a.ml, a.O, a.nsplit, a.c);
}

}  // namespace bb
