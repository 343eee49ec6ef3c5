// rows_kernels_f64.hip -- instantiations of the whole-row scalar kernel, float64 fields.
#include "rows_launch.hpp"

namespace lat {

template hipError_t launch_rows<double, 1>(int, int, int, int, int, const ScalarArgs<double> &, int, hipStream_t, int);
template hipError_t launch_rows<double, 2>(int, int, int, int, int, const ScalarArgs<double> &, int, hipStream_t, int);

}  // namespace lat
