// plane_launch.hpp -- launcher of the any-N plane-run scalar kernel
// (stage_plane.hpp), instantiated per precision in plane_kernels_f64.hip and
// plane_kernels_f32.hip.
#pragma once
#include "launch.hpp"
#include "stage_plane.hpp"

namespace lat {

template <typename T, int NF, int NT, int XS, int HPT, bool DLOAD, bool DEND, bool RED, bool WPHI, bool WPI, int PF>
hipError_t launch_plane_one(const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    const size_t lds = (size_t)2 * NF * (a.tiles_y + 2 * a.N) * sizeof(T);
    const auto fn = scalar_plane<T, NF, NT, XS, HPT, DLOAD, DEND, RED, WPHI, WPI, PF>;
    if (lds > 48 * 1024) {   // beyond what a launch gets by default (with the static part); a constant, so
                             // that calls of several threads agree
        const hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn, dim3(nb), dim3(NT), lds, s, a);
    return hipGetLastError();
}

template <typename T, int NF, int NT, int XS, int HPT, int PF>
hipError_t launch_plane_variant(int variant, const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    switch (variant) {
    case kKickOnly: return launch_plane_one<T, NF, NT, XS, HPT, false, false, false, false, true, PF>(a, nb, s);
    case kKickOnlyRed: return launch_plane_one<T, NF, NT, XS, HPT, false, false, true, false, true, PF>(a, nb, s);
    case kDriftKickRed: return launch_plane_one<T, NF, NT, XS, HPT, true, false, true, true, true, PF>(a, nb, s);
    case kKickDrift: return launch_plane_one<T, NF, NT, XS, HPT, false, true, false, true, true, PF>(a, nb, s);
    case kKickCopy: return launch_plane_one<T, NF, NT, XS, HPT, false, false, false, true, true, PF>(a, nb, s);
    case kKickCopyRed: return launch_plane_one<T, NF, NT, XS, HPT, false, false, true, true, true, PF>(a, nb, s);
    case kEnergy: return launch_plane_one<T, NF, NT, XS, HPT, false, false, true, false, false, PF>(a, nb, s);
    }
    return hipErrorInvalidValue;
}

template <typename T, int NF>
hipError_t launch_plane(const PlaneCfg &c, int variant, const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    // every access stays inside the run, its halo and the plane
    const int NN = a.N * a.N;
    if (a.tiles_y < 1 || a.tiles_y > c.nt * c.xs || 2 * a.N > c.nt * c.hpt || (long)a.tiles_x * a.tiles_y < NN ||
        (long)(a.tiles_x - 1) * a.tiles_y >= NN || a.zc < 1 || nb != a.tiles_x * ((a.N + a.zc - 1) / a.zc))
        return hipErrorInvalidValue;
#define PLANE(NT, XS, HPT)                                                     \
    if (c.nt == NT && c.xs == XS && c.hpt == HPT && c.pf == 1)                 \
        return launch_plane_variant<T, NF, NT, XS, HPT, 1>(variant, a, nb, s);
    PLANE(256, 2, 1)
    if constexpr (sizeof(T) == 8) {
        PLANE(512, 2, 1)
        if constexpr (NF == 1) {
            PLANE(512, 4, 2)
            PLANE(512, 4, 4)
        } else {
            PLANE(512, 2, 2)
            PLANE(512, 2, 4)
        }
    } else {
        PLANE(512, 4, 1)
        PLANE(512, 4, 2)
        PLANE(512, 4, 4)
    }
#undef PLANE
    return hipErrorInvalidValue;
}

}  // namespace lat
