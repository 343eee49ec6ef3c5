// plane_kernels_f64.hip -- instantiations of the plane-run scalar kernel, float64 fields.
#include "plane_launch.hpp"

namespace lat {

template hipError_t launch_plane<double, 1>(const PlaneCfg &, int, const ScalarArgs<double> &, int, hipStream_t);
template hipError_t launch_plane<double, 2>(const PlaneCfg &, int, const ScalarArgs<double> &, int, hipStream_t);

}  // namespace lat
