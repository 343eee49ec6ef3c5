// pair_kernels.hip -- launches of the two-passes-in-one scalar kernel (stage_pair.hpp).
#include "stage_pair.hpp"

namespace lat {

template <typename T, int NF, int XS, int HPT>
static hipError_t launch_pair_one(const PairArgs<T> &a, int nb, hipStream_t s)
{
    const size_t lds = (size_t)NF * (2 * (size_t)(a.seg + 4 * a.N) + 2 * (size_t)(a.seg + 2 * a.N)) * sizeof(T);
    if (lds > kPairLds) return hipErrorInvalidValue;
    const auto fn = scalar_pair<T, NF, XS, HPT>;
    const hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, kPairLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3(nb), dim3(kPairThreads), lds, s, a);
    return hipGetLastError();
}

template <typename T, int NF>
hipError_t launch_pair(int xs, const PairArgs<T> &a, int nb, hipStream_t s)
{
    // every access stays inside the widened run, its neighbours and the plane
    const int NN = a.N * a.N;
    if (a.N < 4 || a.seg < 1 || a.seg + 2 * a.N > kPairThreads * xs || a.seg + 4 * a.N > NN || 2 * a.N > 2 * kPairThreads ||
        (long)a.runs * a.seg < NN || (long)(a.runs - 1) * a.seg >= NN || a.zc < 1 ||
        nb != a.runs * ((a.N + a.zc - 1) / a.zc))
        return hipErrorInvalidValue;
    const bool wide = 2 * a.N > kPairThreads;
#define PAIR(XS) \
    if (xs == XS) return wide ? launch_pair_one<T, NF, XS, 2>(a, nb, s) : launch_pair_one<T, NF, XS, 1>(a, nb, s);
    if constexpr (NF == 1 && sizeof(T) == 8) {
        PAIR(6)
        PAIR(8)
    } else if constexpr (NF == 1) {
        PAIR(8)
        PAIR(12)
    } else if constexpr (sizeof(T) == 8) {
        PAIR(3)
        PAIR(4)
    } else {
        PAIR(6)
    }
#undef PAIR
    return hipErrorInvalidValue;
}

template hipError_t launch_pair<double, 1>(int, const PairArgs<double> &, int, hipStream_t);
template hipError_t launch_pair<double, 2>(int, const PairArgs<double> &, int, hipStream_t);
template hipError_t launch_pair<float, 1>(int, const PairArgs<float> &, int, hipStream_t);
template hipError_t launch_pair<float, 2>(int, const PairArgs<float> &, int, hipStream_t);

}  // namespace lat
