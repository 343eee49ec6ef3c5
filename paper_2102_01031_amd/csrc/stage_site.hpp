// stage_site.hpp -- the stencil pass of stage_scalar.hpp with one site per
// thread: no LDS, no march, every load of a site issued at once.
//
// Thread t of a block owns the sites base + t, base + t + NT, ... of its
// block's run of the linear index n = x + N (y + N z) and loads all stencil
// points of a site itself.  The x neighbours come from the same cache lines,
// the y and z neighbours from lines that other wavefronts of the same XCD have
// loaded (blocks are dealt to the XCDs in runs of whole planes), so while the
// pass's arrays are held in the caches the repeated loads cost little, and the
// marching kernels' serial chain (a load, a barrier and an LDS read per plane)
// is gone.  With several sites per thread the loads of a site are issued
// before the arithmetic of the one before it.
// Bound by the launch (2.7 us back to back) up to 40^3 and by the caches above,
// where the kick-and-drift pass moves its four arrays at 5.5 to 8 TB/s: against the
// marching kernels, two float64 fields 16^3 4.1 -> 2.8 us, 40^3 6.5 -> 3.0,
// 96^3 16.2 -> 12.2; two float32 fields 96^3 13.6 -> 6.2, 160^3 24.9 -> 20.5.  A self-consistent pass reads the momenta at all seven points too
// and begins with the sums of the pass before: 16^3 7.6 -> 6.3 us, 48^3 10.6 -> 8.5.
#pragma once
#include "common.hpp"
#include "stage_scalar.hpp"

namespace lat {

// Reducing passes: ScalarArgs::zc sites per thread, a block's run being zc NT
// sites; the others one site per thread.  Offsets are 32-bit byte offsets: N^3 sizeof(T) < 2^32.
template <typename T, int NF, int NT, bool DLOAD, bool DEND, bool RED, bool WPHI, bool WPI>
__global__ void __launch_bounds__(NT) scalar_site(const ScalarArgs<T> g)
{
    constexpr int NQ = 3 * NF;
    __shared__ double lds_red[RED ? (NT / 64) * NQ : 1];
    __shared__ int last_flag;

    const unsigned N = (unsigned)g.N, NN = N * N, V = NN * N;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const unsigned per = RED ? (unsigned)g.zc : 1u;
    const unsigned base = (unsigned)lid * (per * NT) + threadIdx.x;

    // the stencil points of one site as stored: centre, x -+, y -+, z -+
    struct Raw {
        T f[NF][7], p[NF][DLOAD ? 7 : 1];
    };
    auto load = [&](const unsigned n, Raw &r) {
        const unsigned yz = n / N, x = n - yz * N, z = yz / N, y = yz - z * N;
        const unsigned o[7] = {n,
                               x == 0 ? n + (N - 1) : n - 1,
                               x == N - 1 ? n - (N - 1) : n + 1,
                               y == 0 ? n + (NN - N) : n - N,
                               y == N - 1 ? n - (NN - N) : n + N,
                               z == 0 ? n + (V - NN) : n - NN,
                               z == N - 1 ? n - (V - NN) : n + NN};
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int k = 0; k < 7; ++k) r.f[f][k] = ld32(g.phi_in[f], o[k]);
#pragma unroll
            for (int k = 0; k < (DLOAD ? 7 : 1); ++k) r.p[f][k] = ld32(g.pi_in[f], o[k]);
        }
    };

    Raw r;
    if (base < V) load(base, r);   // issued before the prologue's sums

    PassCoef C = g.by_value ? g.imm : *g.coef;
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

    double acc[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) acc[k] = 0.0;

    auto site = [&](const unsigned n, const Raw &r) {
        T c0[NF], lap[NF], dV[NF];
        T up[NF][3];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            T v[7];
#pragma unroll
            for (int k = 0; k < 7; ++k) v[k] = DLOAD ? r.f[f][k] + dl * r.p[f][DLOAD ? k : 0] : r.f[f][k];
            c0[f] = v[0];
            up[f][0] = v[2];
            up[f][1] = v[4];
            up[f][2] = v[6];
            lap[f] = ((v[2] - T(2) * v[0] + v[1]) + (v[4] - T(2) * v[0] + v[3]) + (v[6] - T(2) * v[0] + v[5])) * idx2;
        }
        if constexpr (NF == 1) {
            const T u = c0[0];
            dV[0] = lam * u * u * u;
        } else {
            const T u = c0[0], w = c0[1];
            dV[0] = lam * u * u * u + qc * u * w * w;
            dV[1] = qc * u * u * w;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const T F = ka1 * lap[f] - ka3 * dV[f];
            const T pm = r.p[f][0] + c1 * F;
            if constexpr (RED) {
                const double pmd = (double)pm;
                acc[f] += pmd * pmd;
                const double gx = (double)(up[f][0] - c0[f]), gy = (double)(up[f][1] - c0[f]),
                             gz = (double)(up[f][2] - c0[f]);
                acc[NF + f] += gx * gx + gy * gy + gz * gz;
            }
            if constexpr (DLOAD) {
                if (g.pi_mid[f]) st32(g.pi_mid[f], n, pm);
            }
            const T pn = pm + c2 * F;
            if (WPHI) st32(g.phi_out[f], n, DEND ? c0[f] + de * pn : c0[f]);
            if (WPI) st32(g.pi_out[f], n, pn);
        }
        if constexpr (RED) {
            const double u = (double)c0[0];
            acc[2 * NF] += 0.25 * lamd * u * u * u * u;
            if constexpr (NF == 2) {
                const double w = (double)c0[1];
                acc[2 * NF + 1] += 0.5 * qd * u * u * w * w;
            }
        }
    };

    if constexpr (!RED) {
        if (base < V) site(base, r);
    } else {
        unsigned n = base;
        for (unsigned k = 0; k < per && n < V; k += 2) {
            Raw s;
            const unsigned n1 = n + NT;
            const bool have1 = k + 1 < per && n1 < V;
            if (have1) load(n1, s);
            site(n, r);
            n = n1 + NT;
            if (k + 2 < per && n < V) load(n, r);
            if (have1) site(n1, s);
        }
    }

    if constexpr (RED) reduce_tail<NT, NF>(g, C, acc, lds_red, &last_flag, lid);
}

}  // namespace lat
