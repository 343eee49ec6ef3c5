// plane_kernels_f32.hip -- instantiations of the plane-run scalar kernel, float32 fields.
#include "plane_launch.hpp"

namespace lat {

template hipError_t launch_plane<float, 1>(const PlaneCfg &, int, const ScalarArgs<float> &, int, hipStream_t);
template hipError_t launch_plane<float, 2>(const PlaneCfg &, int, const ScalarArgs<float> &, int, hipStream_t);

}  // namespace lat
