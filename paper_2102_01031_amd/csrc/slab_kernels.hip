// slab_kernels.hip -- instantiations of the several-steps-per-launch leapfrog
// kernel for small lattices (stage_slab.hpp).
#include "launch.hpp"
#include "stage_slab.hpp"

namespace lat {

template <typename T, int NF, int S, int ZS>
void slab_kernel_of(const void **fn, size_t *lds, int N, int yb)
{
    *fn = (const void *)lf_slab<T, NF, S, ZS>;
    *lds = slab_lds<T, NF, S, ZS>(N, yb);
}

template <typename T, int NF, int S>
bool slab_pick_zs(int zs, const void **fn, size_t *lds, int N, int yb)
{
    switch (zs) {
    case 1: slab_kernel_of<T, NF, S, 1>(fn, lds, N, yb); return true;
    case 2: slab_kernel_of<T, NF, S, 2>(fn, lds, N, yb); return true;
    default: return false;
    }
}

template <typename T, int NF>
bool slab_pick(int S, int zs, const void **fn, size_t *lds, int N, int yb)
{
    switch (S) {
    case 2: return slab_pick_zs<T, NF, 2>(zs, fn, lds, N, yb);
    case 3: return slab_pick_zs<T, NF, 3>(zs, fn, lds, N, yb);
    case 4: return slab_pick_zs<T, NF, 4>(zs, fn, lds, N, yb);
    case 5: return slab_pick_zs<T, NF, 5>(zs, fn, lds, N, yb);
    default: return false;
    }
}

template bool slab_pick<double, 1>(int, int, const void **, size_t *, int, int);
template bool slab_pick<double, 2>(int, int, const void **, size_t *, int, int);
template bool slab_pick<float, 1>(int, int, const void **, size_t *, int, int);
template bool slab_pick<float, 2>(int, int, const void **, size_t *, int, int);

}  // namespace lat
