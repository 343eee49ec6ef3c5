// stage_pair.hpp -- two kick-and-drift passes on a known background in one march:
// temporal blocking for lattices whose passes stream from memory.
//
// The run-and-march layout of stage_plane.hpp (a block owns `seg` consecutive sites of
// the xy plane and marches them through a z chunk), on a run widened by N sites on
// either side: N sites below and above a site hold its in-plane neighbours, so after
// the first pass on the widened run the second pass has what it needs on the block's own
// sites.  Per plane p of the march: the first pass at p (its in-plane neighbours from
// LDS, its z neighbours from registers), its phi to a second LDS plane, then the second
// pass at p - 1, one barrier in all.  The widened sites are advanced redundantly, by
// the same expressions as their owners, so the result is that of two passes, to the
// rounding of products that the compiler fuses in one kernel and not in the other.  Every array is read and written once for two passes (the widened part from
// L2); momenta are read beyond the own sites and so go to the other buffer too.
// Bound by LDS and the vector unit about as much as by memory: 63 KB (float32, one field,
// N = 203) to 156 KB (float64, two fields, N = 506) of LDS, and as a rule a grid of one
// block of 512 threads per CU.  384^3, one float64 field: 1.86 GB at 5.1 TB/s.  Leapfrog step, single passes and pairs: one float64
// field 384^3 347 -> 175 us, 256^3 110 -> 62, 128^3 16.7 -> 15.1; two 256^3 187 -> 113,
// 320^3 403 -> 238, 110^3 19.6 -> 17.4; float32, two fields 384^3 366 -> 187, one 256^3
// 44 -> 36.
#pragma once
#include "common.hpp"
#include "launch.hpp"

namespace lat {


// XS sites per thread cover the widened run, HPT its outer neighbours (2 N <= HPT NT)
template <typename T, int NF, int XS, int HPT>
__global__ void __launch_bounds__(kPairThreads) scalar_pair(const PairArgs<T> g)
{
    constexpr int NT = kPairThreads;
    extern __shared__ __attribute__((aligned(16))) unsigned char pair_lds_raw[];
    const int tid = threadIdx.x;
    const int N = g.N, NN = N * N;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int bs = lid % g.runs, bz = lid / g.runs;   // run fastest: neighbouring runs share an L2
    const int s0 = bs * g.seg, s1 = min(s0 + g.seg, NN), len = s1 - s0, ext = len + 2 * N;
    const int z0 = bz * g.zc, z1 = min(z0 + g.zc, N), zn = z1 - z0;
    // start of plane z0 + k, k = -2 .. zn + 1 (N >= 2)
    auto pl = [&](const int k) {
        int z = z0 + k;
        if (z < 0) z += N;
        if (z >= N) z -= N;
        return (size_t)z * (size_t)NN;
    };
    // LDS: phi of two planes on the widened run and its outer neighbours, then the first
    // pass's phi of two planes on the widened run
    const int pitch0 = g.seg + 4 * N, pitch1 = g.seg + 2 * N;
    T *const B0 = (T *)pair_lds_raw, *const B1 = B0 + 2 * NF * pitch0;
    auto L0 = [&](int buf, int f) { return B0 + (buf * NF + f) * pitch0; };
    auto L1 = [&](int buf, int f) { return B1 + (buf * NF + f) * pitch1; };

    unsigned off[XS];
    int el[XS];          // place on the widened run (a thread past its end repeats the last one)
    bool on[XS], in[XS], x0[XS], x1[XS];
#pragma unroll
    for (int k = 0; k < XS; ++k) {
        const int e = tid + NT * k;
        on[k] = e < ext;
        el[k] = on[k] ? e : ext - 1;
        in[k] = on[k] && e >= N && e < N + len;
        int p = s0 - N + el[k];
        if (p < 0) p += NN;
        if (p >= NN) p -= NN;
        off[k] = (unsigned)p;
        const int x = p % N;
        x0[k] = x == 0;
        x1[k] = x == N - 1;
    }
    unsigned hoff[HPT];
    int hsl[HPT];
    bool hon[HPT];
#pragma unroll
    for (int j = 0; j < HPT; ++j) {
        const int h = tid + NT * j;
        hon[j] = h < 2 * N;
        int q = h < N ? s0 - 2 * N + h : s1 + h;
        if (q < 0) q += NN;
        if (q >= NN) q -= NN;
        hoff[j] = hon[j] ? (unsigned)q : 0u;
        hsl[j] = h < N ? h : ext + h;
    }

    // phi at planes p - 1, p, p + 1 and pi at p; the first pass's phi at p - 2 and p - 1
    // and its pi at p - 1; the outer neighbours' phi at p + 1
    T fm[XS][NF], f0[XS][NF], fp[XS][NF], p0[XS][NF], gm[XS][NF], g0[XS][NF], q0[XS][NF], hc[HPT][NF];
    {
        const size_t om = pl(-2), o0 = pl(-1), o1 = pl(0);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const T *P = g.phi_in[f], *Q = g.pi_in[f];
            T h0[HPT];
#pragma unroll
            for (int k = 0; k < XS; ++k) {
                fm[k][f] = ld32(P + om, off[k]);
                f0[k][f] = ld32(P + o0, off[k]);
                fp[k][f] = ld32(P + o1, off[k]);
                p0[k][f] = ld32(Q + o0, off[k]);
                gm[k][f] = g0[k][f] = q0[k][f] = T(0);
            }
#pragma unroll
            for (int j = 0; j < HPT; ++j) {
                h0[j] = hc[j][f] = T(0);
                if (hon[j]) {
                    h0[j] = ld32(P + o0, hoff[j]);
                    hc[j][f] = ld32(P + o1, hoff[j]);
                }
            }
#pragma unroll
            for (int k = 0; k < XS; ++k) L0(0, f)[N + el[k]] = f0[k][f];
#pragma unroll
            for (int j = 0; j < HPT; ++j)
                if (hon[j]) L0(0, f)[hsl[j]] = h0[j];
        }
    }
    const PassCoef A = g.coef[0], B = g.coef[1];
    const T idx2 = (T)g.inv_dx2, lam = (T)g.lam, qc = (T)g.q;
    const T ac1 = (T)A.c1, ac2 = (T)A.c2, ade = (T)A.dend, aka1 = (T)A.ka1, aka3 = (T)A.ka3;
    const T bc1 = (T)B.c1, bc2 = (T)B.c2, bde = (T)B.dend, bka1 = (T)B.ka1, bka3 = (T)B.ka3;
    __syncthreads();

    // kick and drift of one site: u the fields, lap their Laplacians, pv in: momenta, out:
    // kicked; un out: the drifted fields
    auto advance = [&](const T (&u)[NF], const T (&lap)[NF], T (&pv)[NF], T (&un)[NF], T c1, T c2, T de, T ka1, T ka3) {
        T dV[NF];
        if constexpr (NF == 1) {
            dV[0] = lam * u[0] * u[0] * u[0];
        } else {
            dV[0] = lam * u[0] * u[0] * u[0] + qc * u[0] * u[1] * u[1];
            dV[1] = qc * u[0] * u[0] * u[1];
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const T F = ka1 * lap[f] - ka3 * dV[f];
            const T pm = pv[f] + c1 * F;
            pv[f] = pm + c2 * F;
            un[f] = de != T(0) ? u[f] + de * pv[f] : u[f];   // a closing kick leaves the field as it is
        }
    };

    for (int k = 0; k < zn + 2; ++k) {   // p = z0 - 1 + k
        const int cur = k & 1, nxt = cur ^ 1;
        // plane p + 2 (and its outer neighbours) and pi of p + 1, used in the next round
        T nf[XS][NF], np[XS][NF], hn[HPT][NF];
        {
            const size_t o2 = pl(min(k + 1, zn + 1)), o1 = pl(min(k, zn));
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T *P = g.phi_in[f] + o2, *Q = g.pi_in[f] + o1;
#pragma unroll
                for (int i = 0; i < XS; ++i) {
                    nf[i][f] = ld32(P, off[i]);
                    np[i][f] = ld32(Q, off[i]);
                }
#pragma unroll
                for (int j = 0; j < HPT; ++j) {
                    hn[j][f] = T(0);
                    if (hon[j]) hn[j][f] = ld32(P, hoff[j]);
                }
            }
        }
        // phi of plane p + 1 to LDS
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            T *L = L0(nxt, f);
#pragma unroll
            for (int i = 0; i < XS; ++i) L[N + el[i]] = fp[i][f];
#pragma unroll
            for (int j = 0; j < HPT; ++j)
                if (hon[j]) L[hsl[j]] = hc[j][f];
        }
        const size_t oz = pl(k >= 2 ? k - 2 : 0);
#pragma unroll
        for (int i = 0; i < XS; ++i) {
            const int dm = x0[i] ? N - 1 : -1, dp = x1[i] ? 1 - N : 1;
            // first pass at p
            T u[NF], lap[NF], g1[NF], q1[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const T *L = L0(cur, f) + N + el[i];
                const T c0 = f0[i][f];
                u[f] = c0;
                q1[f] = p0[i][f];
                lap[f] = ((L[dp] - T(2) * c0 + L[dm]) + (L[N] - T(2) * c0 + L[-N]) +
                          (fp[i][f] - T(2) * c0 + fm[i][f])) * idx2;
            }
            advance(u, lap, q1, g1, ac1, ac2, ade, aka1, aka3);
#pragma unroll
            for (int f = 0; f < NF; ++f) L1(cur, f)[el[i]] = g1[f];
            // second pass at p - 1
            if (k >= 2 && in[i]) {
                T un[NF], pv[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const T *L = L1(nxt, f) + el[i];
                    const T c0 = g0[i][f];
                    u[f] = c0;
                    pv[f] = q0[i][f];
                    lap[f] = ((L[dp] - T(2) * c0 + L[dm]) + (L[N] - T(2) * c0 + L[-N]) +
                              (g1[f] - T(2) * c0 + gm[i][f])) * idx2;
                }
                advance(u, lap, pv, un, bc1, bc2, bde, bka1, bka3);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    st32(g.phi_out[f] + oz, off[i], un[f]);
                    st32(g.pi_out[f] + oz, off[i], pv[f]);
                }
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                gm[i][f] = g0[i][f];
                g0[i][f] = g1[f];
                q0[i][f] = q1[f];
                fm[i][f] = f0[i][f];
                f0[i][f] = fp[i][f];
            }
        }
        __syncthreads();
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int i = 0; i < XS; ++i) {
                fp[i][f] = nf[i][f];
                p0[i][f] = np[i][f];
            }
#pragma unroll
            for (int j = 0; j < HPT; ++j) hc[j][f] = hn[j][f];
        }
    }
}

}  // namespace lat
