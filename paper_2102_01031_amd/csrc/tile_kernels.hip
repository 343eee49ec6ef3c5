// tile_kernels.hip -- instantiations of the tiled scalar kernel (stage_scalar.hpp).
#include "launch.hpp"

namespace lat {

template <typename T, int NF, int TX, int TY>
hipError_t launch_variant(int variant, const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    const dim3 grid(nb), block(TX * TY);
    switch (variant) {
    case kKickOnly:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, false, false, false, false, true>), grid, block, 0, s, a);
        break;
    case kKickOnlyRed:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, false, false, true, false, true>), grid, block, 0, s, a);
        break;
    case kDriftKickRed:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, true, false, true, true, true>), grid, block, 0, s, a);
        break;
    case kKickDrift:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, false, true, false, true, true>), grid, block, 0, s, a);
        break;
    case kKickCopy:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, false, false, false, true, true>), grid, block, 0, s, a);
        break;
    case kKickCopyRed:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, false, false, true, true, true>), grid, block, 0, s, a);
        break;
    case kEnergy:
        hipLaunchKernelGGL((scalar_stage<T, NF, TX, TY, false, false, true, false, false>), grid, block, 0, s, a);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, int NF>
hipError_t launch_tile(int tile, int variant, const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    switch (tile) {
    case 0: return launch_variant<T, NF, 64, 4>(variant, a, nb, s);
    case 1: return launch_variant<T, NF, 64, 8>(variant, a, nb, s);
    case 2: return launch_variant<T, NF, 32, 8>(variant, a, nb, s);
    case 3: return launch_variant<T, NF, 16, 16>(variant, a, nb, s);
    case 4: return launch_variant<T, NF, 8, 8>(variant, a, nb, s);
    }
    return hipErrorInvalidValue;
}

template hipError_t launch_tile<double, 1>(int, int, const ScalarArgs<double> &, int, hipStream_t);
template hipError_t launch_tile<double, 2>(int, int, const ScalarArgs<double> &, int, hipStream_t);
template hipError_t launch_tile<float, 1>(int, int, const ScalarArgs<float> &, int, hipStream_t);
template hipError_t launch_tile<float, 2>(int, int, const ScalarArgs<float> &, int, hipStream_t);

}  // namespace lat
