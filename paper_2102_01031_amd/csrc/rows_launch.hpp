// rows_launch.hpp -- launcher of the whole-row scalar kernel (stage_rows.hpp),
// instantiated per precision in rows_kernels_f64.hip and rows_kernels_f32.hip.
#pragma once
#include "launch.hpp"
#include "stage_rows.hpp"

namespace lat {

template <typename T, int NF, int XS, int TY, int PF = 1, int VW = 1, int LP = 0>
hipError_t launch_rows_variant(int variant, const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    const dim3 grid(nb), block(64 * TY);
    switch (variant) {
    case kKickOnly:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, false, false, false, false, true, PF, VW, LP>), grid, block, 0, s, a);
        break;
    case kKickOnlyRed:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, false, false, true, false, true, PF, VW, LP>), grid, block, 0, s, a);
        break;
    case kDriftKickRed:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, true, false, true, true, true, PF, VW, LP>), grid, block, 0, s, a);
        break;
    case kKickDrift:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, false, true, false, true, true, PF, VW, LP>), grid, block, 0, s, a);
        break;
    case kKickCopy:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, false, false, false, true, true, PF, VW, LP>), grid, block, 0, s, a);
        break;
    case kKickCopyRed:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, false, false, true, true, true, PF, VW, LP>), grid, block, 0, s, a);
        break;
    case kEnergy:
        hipLaunchKernelGGL((scalar_rows<T, NF, XS, TY, false, false, true, false, false, PF, VW, LP>), grid, block, 0, s, a);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// pf: prefetch depth in planes (2 is instantiated for N = 256 with 4-row
// blocks only; 8-row float64 blocks would spill at that depth).
// vw > 1: 16-byte accesses (two float64 or four float32 sites per lane and
// access), instantiated where the row holds a whole number of them per lane:
// N = 128, 256 in float64, N = 256 in float32.
// lp: store policy of the row kernel (RowPolicy in stage_rows.hpp; 1 streams
// the first part of the march past the caches), instantiated for the N = 256
// defaults (float64 4-row blocks two planes ahead, float32 4-row blocks four
// planes ahead with 16-byte accesses); elsewhere policy 0.
template <typename T, int NF>
hipError_t launch_rows(int N, int ty, int pf, int vw, int variant, const ScalarArgs<T> &a, int nb, hipStream_t s,
                       int lp)
{
    const int xs = N / 64;
    constexpr int V = 16 / (int)sizeof(T);
    if constexpr (sizeof(T) == 8) {
        if (lp == 1 && vw == 1 && pf == 2 && xs == 4 && ty == 4)
            return launch_rows_variant<T, NF, 4, 4, 2, 1, 1>(variant, a, nb, s);
    } else {
        if (lp == 1 && vw > 1 && pf == 4 && xs == 4 && ty == 4)
            return launch_rows_variant<T, NF, 4, 4, 4, V, 1>(variant, a, nb, s);
    }
    if (vw > 1 && xs % V == 0) {
        if (pf == 2 && xs == 4 && ty == 4) return launch_rows_variant<T, NF, 4, 4, 2, V>(variant, a, nb, s);
        if constexpr (V == 4) {
            if (pf == 2 && xs == 4 && ty == 8) return launch_rows_variant<T, NF, 4, 8, 2, V>(variant, a, nb, s);
            if (pf == 3 && xs == 4 && ty == 4) return launch_rows_variant<T, NF, 4, 4, 3, V>(variant, a, nb, s);
            if (pf == 4 && xs == 4 && ty == 4) return launch_rows_variant<T, NF, 4, 4, 4, V>(variant, a, nb, s);
        }
        if (xs == 4) return ty == 4 ? launch_rows_variant<T, NF, 4, 4, 1, V>(variant, a, nb, s)
                                    : launch_rows_variant<T, NF, 4, 8, 1, V>(variant, a, nb, s);
        if constexpr (V == 2) {
            if (xs == 2) return ty == 4 ? launch_rows_variant<T, NF, 2, 4, 1, V>(variant, a, nb, s)
                                        : launch_rows_variant<T, NF, 2, 8, 1, V>(variant, a, nb, s);
        }
        return hipErrorInvalidValue;
    }
    if (pf == 2 && xs == 4 && ty == 4) return launch_rows_variant<T, NF, 4, 4, 2>(variant, a, nb, s);
    if constexpr (sizeof(T) == 8) {
        if (pf == 3 && xs == 4 && ty == 4) return launch_rows_variant<T, NF, 4, 4, 3>(variant, a, nb, s);
    }
    if (ty == 4) {
        if (xs == 1) return launch_rows_variant<T, NF, 1, 4>(variant, a, nb, s);
        if (xs == 2) return launch_rows_variant<T, NF, 2, 4>(variant, a, nb, s);
        if (xs == 4) return launch_rows_variant<T, NF, 4, 4>(variant, a, nb, s);
    } else {
        if (xs == 1) return launch_rows_variant<T, NF, 1, 8>(variant, a, nb, s);
        if (xs == 2) return launch_rows_variant<T, NF, 2, 8>(variant, a, nb, s);
        if (xs == 4) return launch_rows_variant<T, NF, 4, 8>(variant, a, nb, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace lat
