// rows_kernels_f32.hip -- instantiations of the whole-row scalar kernel, float32 fields.
#include "rows_launch.hpp"

namespace lat {

template hipError_t launch_rows<float, 1>(int, int, int, int, int, const ScalarArgs<float> &, int, hipStream_t, int);
template hipError_t launch_rows<float, 2>(int, int, int, int, int, const ScalarArgs<float> &, int, hipStream_t, int);

}  // namespace lat
