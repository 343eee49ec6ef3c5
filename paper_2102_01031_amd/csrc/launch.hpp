// launch.hpp -- kernel launchers of the real scalar passes, each compiled in a
// translation unit of its own (tile_kernels.hip, rows_kernels_*.hip,
// plane_kernels_*.hip, slab_kernels.hip), so that the instantiations build in
// parallel.
#pragma once
#include "common.hpp"
#include "stage_scalar.hpp"

namespace lat {

struct TileCfg {
    int tx, ty;
};
constexpr TileCfg kTiles[] = {{64, 4}, {64, 8}, {32, 8}, {16, 16}, {8, 8}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

enum Variant : int {
    kKickOnly = 0,     // no drift, kick, momenta in place (VV first point, LF sync)
    kKickOnlyRed = 1,  // same + reductions (self-consistent first point)
    kDriftKickRed = 3, // drift on load, kick + reductions (self-consistent)
    kKickDrift = 4,    // kick, drift at end (leapfrog; VV sub-steps on a known background)
    kEnergy = 5,       // kick on a copy + reductions, writes nothing
    kKickCopy = 6,     // kick only, phi carried to the other buffer (see step_vv)
    kKickCopyRed = 7   // kick only + reductions, phi and pi written to the other buffers
};

// one pass of the tiled kernel (any N) with tile shape kTiles[tile]
template <typename T, int NF>
hipError_t launch_tile(int tile, int variant, const ScalarArgs<T> &a, int nb, hipStream_t s);

// one pass of the whole-row kernel (N = 64, 128, 256); see rows_launch.hpp
template <typename T, int NF>
hipError_t launch_rows(int N, int ty, int pf, int vw, int variant, const ScalarArgs<T> &a, int nb, hipStream_t s,
                       int lp = 0);

// Launch shape of the plane-run kernel (stage_plane.hpp): threads per block,
// sites and halo sites per thread, prefetch depth.
struct PlaneCfg {
    int nt, xs, hpt, pf;
};
// one pass of the plane-run kernel (any N with 2 N <= hpt nt)
template <typename T, int NF>
hipError_t launch_plane(const PlaneCfg &c, int variant, const ScalarArgs<T> &a, int nb, hipStream_t s);

// one pass of the one-site-per-thread kernel (stage_site.hpp): any N with
// N^3 sizeof(T) < 2^32; blocks of kSiteThreads
constexpr int kSiteThreads = 256;
template <typename T, int NF>
hipError_t launch_site(int variant, const ScalarArgs<T> &a, int nb, hipStream_t s);

// Two kick-and-drift passes in one launch (stage_pair.hpp): runs of seg sites, zc planes
// per block, the coefficients of both passes.  xs: sites per thread of the run widened
// by 2 N; 4 <= N <= 512, and the runs' planes fit kPairLds bytes of LDS.
template <typename T>
struct PairArgs {
    const T *phi_in[2], *pi_in[2];
    T *phi_out[2], *pi_out[2];
    int N, zc, runs, seg;
    double inv_dx2, lam, q;
    const PassCoef *coef;
};
constexpr int kPairLds = 156 * 1024, kPairThreads = 512;
template <typename T, int NF>
hipError_t launch_pair(int xs, const PairArgs<T> &a, int nb, hipStream_t s);

// the lf_slab instance for S steps per launch and ZS planes per block, and its
// dynamic LDS for yb rows per block; false if that shape is not compiled
template <typename T, int NF>
bool slab_pick(int S, int zs, const void **fn, size_t *lds, int N, int yb);

}  // namespace lat
