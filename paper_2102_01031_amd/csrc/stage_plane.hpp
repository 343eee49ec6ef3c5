// stage_plane.hpp -- the stencil pass of stage_scalar.hpp for any N: a block
// owns a run of consecutive sites of the xy plane, whatever the row length.
//
// The N^2 sites of a plane are cut into equal runs of `seg` sites (x fastest,
// rows cut where they fall); a block marches one run through a z chunk.  In
// the plane's linear index p = x + N y the periodic y neighbours are p -+ N
// (mod N^2) and the x neighbours p -+ 1, or p -+ (N - 1) across a row's ends:
// all of them lie within N sites of p, so the run plus N sites below and N
// above, one contiguous piece of LDS, holds every in-plane neighbour.  Thread
// t owns the run's sites t + NT k (k < XS), so each access of a wavefront is
// one contiguous segment for every N, and no thread idles except in the last
// 2 NT XS sites' rounding of the cut (a tile of fixed width leaves up to half
// of its threads without a site where N is not a multiple of the tile).
// z neighbours come from a register window, the loads run PF planes ahead of
// their use, and the reductions and the deferred scale-factor update are those
// of stage_scalar.hpp, as is the arithmetic of a site, term by term.
// Bound by the memory and by the bytes in flight: a pass takes the blocks'
// start-up (three planes' loads, the sums of the pass before) once per round of
// resident blocks, so the cut of the lattice fills one round where it can.
// Measured per self-consistent velocity-Verlet pass of two fields against the
// 8 x 8 tiles that N off a multiple of 16 had before: 135^3 float64 70.6 -> 41.6 us,
// 200^3 float32 171 -> 57 us (4.5 TB/s), 200^3 float64 244 -> 128 us; one float64
// field's leapfrog pass: 135^3 45 -> 17 us, 200^3 109 -> 42 us (6.1 TB/s), 384^3
// (64 x 8 tiles before) 441 -> 349 us (5.2 TB/s).  Non-temporal stores and
// alternating march directions measured the same within 1%.
#pragma once
#include "common.hpp"
#include "stage_scalar.hpp"

namespace lat {

// ScalarArgs::tiles_x runs per plane, ScalarArgs::tiles_y sites per run; HPT: halo
// sites per thread, 2 N <= HPT NT.  LDS: 2 NF (seg + 2 N) values of T.
template <typename T, int NF, int NT, int XS, int HPT, bool DLOAD, bool DEND, bool RED, bool WPHI, bool WPI, int PF>
__global__ void __launch_bounds__(NT) scalar_plane(const ScalarArgs<T> g)
{
    constexpr int NQ = 3 * NF;
    extern __shared__ __attribute__((aligned(16))) unsigned char plane_lds_raw[];
    __shared__ double lds_red[(NT / 64) * NQ];
    __shared__ int last_flag;

    const int tid = threadIdx.x;
    const int N = g.N, NN = N * N, seg = g.tiles_y;
    // run fastest: the blocks of one XCD hold neighbouring runs of the same
    // planes, so the N sites two runs share are read from HBM once
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int bs = lid % g.tiles_x, bz = lid / g.tiles_x;
    const int s0 = bs * seg, s1 = min(s0 + seg, NN), len = s1 - s0;
    const int z0 = bz * g.zc, z1 = min(z0 + g.zc, N), zn = z1 - z0;
    // start of plane z0 + k, k = -1 .. zn
    auto pl = [&](const int k) {
        int z = z0 + k;
        if (z < 0) z += N;
        if (z >= N) z -= N;
        return (size_t)z * (size_t)NN;
    };
    const int pitch = seg + 2 * N;              // LDS values per field and buffer
    T *const L0 = (T *)plane_lds_raw;
    auto LP = [&](int buf, int f) { return L0 + (buf * NF + f) * pitch; };

    // own sites: plane offset, LDS slot and the slots of the x neighbours (a
    // thread without a k-th site repeats the run's last one and stores nothing)
    unsigned off[XS];
    int sl[XS], sxm[XS], sxp[XS];
    bool valid[XS];
#pragma unroll
    for (int k = 0; k < XS; ++k) {
        const int p = s0 + tid + NT * k;
        valid[k] = p < s1;
        const int pc = valid[k] ? p : s1 - 1;
        off[k] = (unsigned)pc;
        sl[k] = N + pc - s0;
        const int x = pc % N;
        sxm[k] = x == 0 ? sl[k] + N - 1 : sl[k] - 1;
        sxp[k] = x == N - 1 ? sl[k] - N + 1 : sl[k] + 1;
    }
    unsigned hoff[HPT];
    int hsl[HPT];
    bool hval[HPT];
#pragma unroll
    for (int j = 0; j < HPT; ++j) {
        const int h = tid + NT * j;
        hval[j] = h < 2 * N;
        int q = h < N ? s0 - N + h : s1 - N + h;
        if (q < 0) q += NN;
        if (q >= NN) q -= NN;
        hoff[j] = hval[j] ? (unsigned)q : 0u;
        hsl[j] = h < N ? h : len + h;
    }

    T fm[XS][NF], f0[XS][NF], fp[XS][NF], p0[XS][NF], pp[XS][NF];
    T of[PF + 1][XS][NF], op[PF + 1][XS][NF], hf[PF + 1][HPT][NF], hp[PF + 1][HPT][NF];
    // planes -1, 0, 1 and the halo of plane 0, raw; sets 0 .. PF-1: own plane
    // 2 + s and halo plane 1 + s.  Issued before the prologue's sums.
    T ra[XS][NF], rpa[XS][NF], rpc[XS][NF], rh[HPT][NF], rph[HPT][NF];
    {
        const size_t om = pl(-1), o0 = pl(0), o1 = pl(1);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const T *P = g.phi_in[f], *Q = g.pi_in[f];
#pragma unroll
            for (int k = 0; k < XS; ++k) {
                ra[k][f] = ld32(P + om, off[k]);
                rpa[k][f] = DLOAD ? ld32(Q + om, off[k]) : T(0);
                f0[k][f] = ld32(P + o0, off[k]);
                p0[k][f] = ld32(Q + o0, off[k]);
                fp[k][f] = ld32(P + o1, off[k]);
                pp[k][f] = ld32(Q + o1, off[k]);
            }
#pragma unroll
            for (int j = 0; j < HPT; ++j) {
                rh[j][f] = rph[j][f] = T(0);
                if (hval[j]) {
                    rh[j][f] = ld32(P + o0, hoff[j]);
                    if (DLOAD) rph[j][f] = ld32(Q + o0, hoff[j]);
                }
            }
#pragma unroll
            for (int s = 0; s < PF; ++s) {
                const size_t os = pl(min(2 + s, zn)), oh = pl(min(1 + s, zn - 1));
#pragma unroll
                for (int k = 0; k < XS; ++k) {
                    of[s][k][f] = ld32(P + os, off[k]);
                    op[s][k][f] = ld32(Q + os, off[k]);
                }
#pragma unroll
                for (int j = 0; j < HPT; ++j) {
                    hf[s][j][f] = hp[s][j][f] = T(0);
                    if (hval[j]) {
                        hf[s][j][f] = ld32(P + oh, hoff[j]);
                        if (DLOAD) hp[s][j][f] = ld32(Q + oh, hoff[j]);
                    }
                }
            }
        }
    }

    PassCoef C = *g.coef;
    if constexpr (RED) {   // the other passes follow no deferring pass
        if (g.fin) {
            __shared__ double lds_coef[4];
            finalise_prologue<NT, NF>(g, lds_red, lds_coef, C);
        }
    }
    const T dl = (T)C.dload, c1 = (T)C.c1, c2 = (T)C.c2, de = (T)C.dend;
    const T ka1 = (T)C.ka1, ka3 = (T)C.ka3, idx2 = (T)g.inv_dx2;
    const T lam = (T)g.lam, qc = (T)g.q;
    const double lamd = g.lam, qd = g.q;

#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
        for (int k = 0; k < XS; ++k) {
            fm[k][f] = DLOAD ? ra[k][f] + dl * rpa[k][f] : ra[k][f];
            if (DLOAD) {
                f0[k][f] += dl * p0[k][f];
                fp[k][f] += dl * pp[k][f];
            }
            LP(0, f)[sl[k]] = f0[k][f];
        }
#pragma unroll
        for (int j = 0; j < HPT; ++j)
            if (hval[j]) LP(0, f)[hsl[j]] = DLOAD ? rh[j][f] + dl * rph[j][f] : rh[j][f];
    }
    __syncthreads();

    double acc[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) acc[k] = 0.0;

    auto plane = [&](const int sm, T (&oif)[XS][NF], T (&oip)[XS][NF], T (&hif)[HPT][NF], T (&hip)[HPT][NF],
                     T (&oof)[XS][NF], T (&oop)[XS][NF], T (&hof)[HPT][NF], T (&hop)[HPT][NF]) {
        const int cur = sm & 1, nxt = cur ^ 1;
        const size_t o3 = pl(min(sm + 2 + PF, zn)), o2 = pl(min(sm + 1 + PF, zn - 1));
        // (A) loads PF planes ahead
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const T *P3 = g.phi_in[f] + o3, *Q3 = g.pi_in[f] + o3, *P2 = g.phi_in[f] + o2, *Q2 = g.pi_in[f] + o2;
#pragma unroll
            for (int k = 0; k < XS; ++k) {
                oof[k][f] = ld32(P3, off[k]);
                oop[k][f] = ld32(Q3, off[k]);
            }
#pragma unroll
            for (int j = 0; j < HPT; ++j) {
                if (hval[j]) {
                    hof[j][f] = ld32(P2, hoff[j]);
                    if (DLOAD) hop[j][f] = ld32(Q2, hoff[j]);
                }
            }
        }
        // (B) LDS: the plane ahead
        if (sm + 1 < zn) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                T *L = LP(nxt, f);
#pragma unroll
                for (int k = 0; k < XS; ++k) L[sl[k]] = fp[k][f];
#pragma unroll
                for (int j = 0; j < HPT; ++j)
                    if (hval[j]) L[hsl[j]] = DLOAD ? hif[j][f] + dl * hip[j][f] : hif[j][f];
            }
        }
        // (C) the XS sites of this thread
        const size_t oz = pl(sm);
#pragma unroll
        for (int k = 0; k < XS; ++k) {
            T xp[NF], yp[NF], zp[NF], lap[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T *L = LP(cur, f);
                const T xm = L[sxm[k]], ym = L[sl[k] - N], c0 = f0[k][f];
                xp[f] = L[sxp[k]];
                yp[f] = L[sl[k] + N];
                zp[f] = fp[k][f];
                const T zm = fm[k][f];
                lap[f] = ((xp[f] - T(2) * c0 + xm) + (yp[f] - T(2) * c0 + ym) + (zp[f] - T(2) * c0 + zm)) * idx2;
            }
            T dV[NF];
            if constexpr (NF == 1) {
                const T u = f0[k][0];
                dV[0] = lam * u * u * u;
            } else {
                const T u = f0[k][0], w = f0[k][1];
                dV[0] = lam * u * u * u + qc * u * w * w;
                dV[1] = qc * u * u * w;
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T F = ka1 * lap[f] - ka3 * dV[f];
                const T pm = p0[k][f] + c1 * F;
                if (RED && valid[k]) {
                    const double pmd = (double)pm;
                    acc[f] += pmd * pmd;
                    const double gx = (double)(xp[f] - f0[k][f]), gy = (double)(yp[f] - f0[k][f]),
                                 gz = (double)(zp[f] - f0[k][f]);
                    acc[NF + f] += gx * gx + gy * gy + gz * gz;
                }
                const T pn = pm + c2 * F;
                const T fo = DEND ? f0[k][f] + de * pn : f0[k][f];
                if (valid[k]) {
                    if (WPHI) st32(g.phi_out[f] + oz, off[k], fo);
                    if (WPI) st32(g.pi_out[f] + oz, off[k], pn);
                }
            }
            if (RED && valid[k]) {
                const double u = (double)f0[k][0];
                acc[2 * NF] += 0.25 * lamd * u * u * u * u;
                if constexpr (NF == 2) {
                    const double w = (double)f0[k][1];
                    acc[2 * NF + 1] += 0.5 * qd * u * u * w * w;
                }
            }
        }
        __syncthreads();
        // (E) rotate the window
#pragma unroll
        for (int k = 0; k < XS; ++k) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                fm[k][f] = f0[k][f];
                f0[k][f] = fp[k][f];
                p0[k][f] = pp[k][f];
                fp[k][f] = DLOAD ? oif[k][f] + dl * oip[k][f] : oif[k][f];
                pp[k][f] = oip[k][f];
            }
        }
    };

    for (int sm = 0; sm < zn; sm += PF + 1) {
#pragma unroll
        for (int u = 0; u <= PF; ++u) {
            if (sm + u < zn) {
                const int d = (u + PF) % (PF + 1);
                plane(sm + u, of[u], op[u], hf[u], hp[u], of[d], op[d], hf[d], hp[d]);
            }
        }
    }

    if constexpr (RED) reduce_tail<NT, NF>(g, C, acc, lds_red, &last_flag, lid);
}

}  // namespace lat
