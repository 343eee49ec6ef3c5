// site_kernels.hip -- instantiations of the one-site-per-thread scalar kernel
// (stage_site.hpp).
#include "launch.hpp"
#include "stage_site.hpp"

namespace lat {

template <typename T, int NF, bool DLOAD, bool DEND, bool RED, bool WPHI, bool WPI>
static hipError_t launch_site_one(const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    hipLaunchKernelGGL((scalar_site<T, NF, kSiteThreads, DLOAD, DEND, RED, WPHI, WPI>), dim3(nb), dim3(kSiteThreads),
                       0, s, a);
    return hipGetLastError();
}

template <typename T, int NF>
hipError_t launch_site(int variant, const ScalarArgs<T> &a, int nb, hipStream_t s)
{
    // the blocks' runs cover the lattice, and its byte offsets fit 32 bits
    const bool red = variant == kKickOnlyRed || variant == kDriftKickRed || variant == kKickCopyRed || variant == kEnergy;
    const double V = (double)a.N * a.N * a.N;
    if (a.N < 1 || (a.fin && !red) || V * sizeof(T) >= 4294967296.0 || (red && a.zc < 1) ||
        (double)nb * kSiteThreads * (red ? a.zc : 1) < V || (double)nb * kSiteThreads * (red ? a.zc : 1) >= 4294967296.0)
        return hipErrorInvalidValue;
    switch (variant) {
    case kKickOnly: return launch_site_one<T, NF, false, false, false, false, true>(a, nb, s);
    case kKickOnlyRed: return launch_site_one<T, NF, false, false, true, false, true>(a, nb, s);
    case kDriftKickRed: return launch_site_one<T, NF, true, false, true, true, true>(a, nb, s);
    case kKickDrift: return launch_site_one<T, NF, false, true, false, true, true>(a, nb, s);
    case kKickCopy: return launch_site_one<T, NF, false, false, false, true, true>(a, nb, s);
    case kKickCopyRed: return launch_site_one<T, NF, false, false, true, true, true>(a, nb, s);
    case kEnergy: return launch_site_one<T, NF, false, false, true, false, false>(a, nb, s);
    }
    return hipErrorInvalidValue;
}

template hipError_t launch_site<double, 1>(int, const ScalarArgs<double> &, int, hipStream_t);
template hipError_t launch_site<double, 2>(int, const ScalarArgs<double> &, int, hipStream_t);
template hipError_t launch_site<float, 1>(int, const ScalarArgs<float> &, int, hipStream_t);
template hipError_t launch_site<float, 2>(int, const ScalarArgs<float> &, int, hipStream_t);

}  // namespace lat
