// stage_u1.hpp -- one pass of the U(1) (Abelian-Higgs) lattice system (the
// forces below at a = 1; in an expanding background each term carries its
// power of a, see U1Args).
//
// Complex scalar phi = (phi0 + i phi1)/sqrt(2) (eq. ChargedScalars); psi = phi0 + i phi1.
// Links V_i(n) = exp(-i e dx A_i(n)); plaquette angle (U(1) toolkit, sec. 3.2)
//   theta_ij(n) = e dx [A_j(n+i) - A_j(n) - A_i(n+j) + A_i(n)],
// so that V_i V_{j,+i} V*_{i,+j} V*_j = exp(-i theta_ij).
// Forces, minus the derivative of the lattice Hamiltonian (sec. 5.5.2 kernels):
//   F_phi0 + i F_phi1 = dx^-2 sum_i [V_i psi(n+i) - 2 psi(n) + V*_i(n-i) psi(n-i)]
//                       - lambda/2 (|phi|^2 - v^2) psi
//   F_A_i = kappa_g J_i - (e dx^3)^-1 sum_{j != i} [sin theta_ij(n) - sin theta_ij(n-j)]
//   J_i   = (e/dx) Im[conj(psi(n)) V_i(n) psi(n+i)]
// Leapfrog pass: kick pi, piA by ck, then drift phi, A by hd (phi and A are read
// with neighbours and written to the other buffer; pi and piA in place).
// Energy pass (read only): momenta half-kicked by ck on the fly; energies
//   E_K^phi = (pi0^2 + pi1^2)/2, E_G^phi = sum_i |V_i psi(n+i) - psi(n)|^2 / (2 dx^2),
//   E_V = lambda/4 (|phi|^2 - v^2)^2, E_K^A = sum_i piA_i^2 / (2 kappa_g),
//   E_G^A = sum_{i<j} 2 sin^2(theta_ij/2) / (kappa_g e^2 dx^4),
// and the Gauss residual of the stored pairing (eq. GaussU1-eom at a = 1)
//   G = sum_i (piA_i(n) - piA_i(n-i))/dx - e kappa_g (phi0 pi1 - phi1 pi0).
#pragma once
#include "common.hpp"
#include "trig.hpp"

namespace lat {

struct U1Args {
    const double *phi_in[2];
    double *phi_out[2];
    double *pi[2];
    const double *A_in[3];
    double *A_out[3];
    double *piA[3];
    int N, tiles_x, tiles_y, zc;
    double dx, e, lam, v, kappa_g;
    double ck;   // kick weight (time)
    double hd;   // drift weight of phi (time times a^{alpha-3})
    // expanding background (sec. 5.5.2 kernels): the covariant Laplacian and the
    // current scale with la1 = a^{1+alpha}, the potential force with
    // la3 = a^{3+alpha}, the magnetic force with lam1 = a^{alpha-1}; hdA is the
    // drift weight of A (time times a^{alpha-1}).  All 1 (hdA = hd) at a = 1.
    double la1, la3, lam1, hdA;
    // if not null: {ck, la1, la3, lam1, hd, hdA, ck2} from device memory (written by
    // the self-consistent scale-factor kernels), in place of the values above
    const double *dw;
    double *partials;
    double ck2;  // a second kick weight, applied after the first (and after the sums of kU1KickSums)
};

// kU1KickSums (u1_span only): kicks by ck, forms the volume sums [0, 5) of that state and
// the momentum sums [8, 10) before the kick, then kicks by ck2 (Gauss terms not
// measured: sums [5, 8) and the maxes are zero).  kU1Kick with output arrays also
// carries psi and A over to them.  kU1Drift: the drift alone (u1_drift).
enum U1Mode : int { kU1Step = 0, kU1Kick = 1, kU1Energy = 2, kU1KickSums = 3, kU1Drift = 4 };
// Volume sums of a summing pass: 0 scalar kinetic, 1 gradient, 2 potential, 3 electric,
// 4 magnetic, 5-7 Gauss means, 8 and 9 the kinetic and electric sums of the momenta
// before the pass's kick; then the Gauss maxima.
constexpr int kU1Sums = 10, kU1Maxes = 3;

// the block's sums and maxima of acc to out (thread 0)
template <int NQ>
__device__ inline void u1_block_sums(double (&acc)[NQ], double *lds_red, double *out)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, nw = blockDim.x / 64;
    double v[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) v[k] = k < kU1Sums ? wave_sum(acc[k]) : wave_max(acc[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NQ; ++k) lds_red[w * NQ + k] = v[k];
    }
    __syncthreads();
    if (tid < NQ) {
        double r = 0.0;
        for (int i = 0; i < nw; ++i) r = tid < kU1Sums ? r + lds_red[i * NQ + tid] : fmax(r, lds_red[i * NQ + tid]);
        out[tid] = r;
    }
}

__device__ inline size_t u1_at(int N, int x, int y, int z)
{
    return (size_t)x + (size_t)N * ((size_t)y + (size_t)N * (size_t)z);
}

template <int TX, int TY, int MODE>
__global__ void __launch_bounds__(TX *TY) u1_stage(const U1Args g)
{
    constexpr int NT = TX * TY;
    constexpr int NQ = kU1Sums + kU1Maxes;
    __shared__ double lds_red[(NT / 64) * NQ];

    const int tid = threadIdx.x;
    const int tx = tid % TX, ty = tid / TX;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int bx = lid % g.tiles_x;
    const int rest = lid / g.tiles_x;
    const int by = rest % g.tiles_y;
    const int N = g.N;
    const int x = bx * TX + tx, y = by * TY + ty;
    const bool valid = x < N && y < N;
    // the energy pass takes a column of zc planes per block (fewer partials for the
    // kernel that adds them up); the other passes one plane
    const int zb = MODE == kU1Energy ? (rest / g.tiles_y) * g.zc : rest / g.tiles_y;
    const int ze = MODE == kU1Energy ? min(zb + g.zc, N) : zb + 1;

    double acc[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) acc[k] = 0.0;

#pragma unroll 1
    for (int z = zb; z < ze; ++z) {
    if (valid) {
        const int xm = x == 0 ? N - 1 : x - 1, xp = x + 1 == N ? 0 : x + 1;
        const int ym = y == 0 ? N - 1 : y - 1, yp = y + 1 == N ? 0 : y + 1;
        const int zm = z == 0 ? N - 1 : z - 1, zp = z + 1 == N ? 0 : z + 1;
        const size_t n = u1_at(N, x, y, z);
        const size_t nxp = u1_at(N, xp, y, z), nxm = u1_at(N, xm, y, z);
        const size_t nyp = u1_at(N, x, yp, z), nym = u1_at(N, x, ym, z);
        const size_t nzp = u1_at(N, x, y, zp), nzm = u1_at(N, x, y, zm);
        const double *Ax = g.A_in[0], *Ay = g.A_in[1], *Az = g.A_in[2];
        const double edx = g.e * g.dx;

        // plaquette angles at n and at n - j
        const double txy = edx * ((Ay[nxp] - Ay[n]) - Ax[nyp] + Ax[n]);
        const double txz = edx * ((Az[nxp] - Az[n]) - Ax[nzp] + Ax[n]);
        const double tyz = edx * ((Az[nyp] - Az[n]) - Ay[nzp] + Ay[n]);
        const double txy_xm = edx * ((Ay[n] - Ay[nxm]) - Ax[u1_at(N, xm, yp, z)] + Ax[nxm]);
        const double txz_xm = edx * ((Az[n] - Az[nxm]) - Ax[u1_at(N, xm, y, zp)] + Ax[nxm]);
        const double txy_ym = edx * ((Ay[u1_at(N, xp, ym, z)] - Ay[nym]) - Ax[n] + Ax[nym]);
        const double tyz_ym = edx * ((Az[n] - Az[nym]) - Ay[u1_at(N, x, ym, zp)] + Ay[nym]);
        const double txz_zm = edx * ((Az[u1_at(N, xp, y, zm)] - Az[nzm]) - Ax[n] + Ax[nzm]);
        const double tyz_zm = edx * ((Az[u1_at(N, x, yp, zm)] - Az[nzm]) - Ay[n] + Ay[nzm]);
        const double sxy = lat_sin(txy), sxz = lat_sin(txz), syz = lat_sin(tyz);
        const double mag[3] = {(sxy - lat_sin(txy_ym)) + (sxz - lat_sin(txz_zm)),
                               (-sxy + lat_sin(txy_xm)) + (syz - lat_sin(tyz_zm)),
                               (-sxz + lat_sin(txz_xm)) + (-syz + lat_sin(tyz_ym))};

        // covariant Laplacian and current
        const double pr = g.phi_in[0][n], pim = g.phi_in[1][n];
        const size_t np_[3] = {nxp, nyp, nzp}, nm_[3] = {nxm, nym, nzm};
        double d2r = 0.0, d2i = 0.0, grad2 = 0.0, J[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double s, c, sm, cm;
            lat_sincos(edx * g.A_in[i][n], &s, &c);
            lat_sincos(edx * g.A_in[i][nm_[i]], &sm, &cm);
            s = -s;   // V_i(n) = c + i s ; conj(V_i(n-i)) = cm + i sm
            const double qr = g.phi_in[0][np_[i]], qi = g.phi_in[1][np_[i]];
            const double rr = g.phi_in[0][nm_[i]], ri = g.phi_in[1][nm_[i]];
            const double ar = c * qr - s * qi, ai = c * qi + s * qr;
            const double br = cm * rr - sm * ri, bi = cm * ri + sm * rr;
            d2r += ar - 2.0 * pr + br;
            d2i += ai - 2.0 * pim + bi;
            J[i] = g.e / g.dx * (pr * ai - pim * ar);
            if (MODE == kU1Energy) {
                const double dr = ar - pr, di = ai - pim;
                grad2 += dr * dr + di * di;
            }
        }
        double ck = g.ck, ck2 = g.ck2, la1 = g.la1, la3 = g.la3, lm1 = g.lam1, hdP = g.hd, hdA = g.hdA;
        if (g.dw) {
            ck = g.dw[0];
            la1 = g.dw[1];
            la3 = g.dw[2];
            lm1 = g.dw[3];
            hdP = g.dw[4];
            hdA = g.dw[5];
            ck2 = g.dw[6];
        }
        const double m2 = 0.5 * (pr * pr + pim * pim);
        const double vp = 0.5 * g.lam * (m2 - g.v * g.v);
        const double inv_dx2 = 1.0 / (g.dx * g.dx);
        const double F0 = la1 * (d2r * inv_dx2) - la3 * (vp * pr);
        const double F1 = la1 * (d2i * inv_dx2) - la3 * (vp * pim);
        const double inv_edx3 = 1.0 / (g.e * g.dx * g.dx * g.dx);
        double FA[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) FA[i] = la1 * (g.kappa_g * J[i]) - lm1 * (mag[i] * inv_edx3);

        const double p0 = g.pi[0][n], p1 = g.pi[1][n];
        double pa[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) pa[i] = g.piA[i][n];

        if (MODE == kU1Energy) {
            double t[NQ];
            const double s0 = p0 + ck * F0, s1 = p1 + ck * F1;
            t[0] = 0.5 * (s0 * s0 + s1 * s1);
            t[1] = grad2 * inv_dx2 * 0.5;
            const double u = m2 - g.v * g.v;
            t[2] = 0.25 * g.lam * u * u;
            double ka = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double sa = pa[i] + ck * FA[i];
                ka += sa * sa;
            }
            t[3] = ka / (2.0 * g.kappa_g);
            const double hxy = lat_sin(0.5 * txy), hxz = lat_sin(0.5 * txz), hyz = lat_sin(0.5 * tyz);
            const double mg = 2.0 * hxy * hxy + 2.0 * hxz * hxz + 2.0 * hyz * hyz;
            t[4] = mg / (g.kappa_g * g.e * g.e * g.dx * g.dx * g.dx * g.dx);
            // Gauss residual of the stored pairing
            const double div = ((pa[0] - g.piA[0][nxm]) + (pa[1] - g.piA[1][nym]) + (pa[2] - g.piA[2][nzm])) / g.dx;
            const double charge = g.e * g.kappa_g * (pr * p1 - pim * p0);
            const double G = div - charge;
            t[5] = fabs(G);
            t[6] = fabs(div + charge);
            t[7] = fabs(div) + fabs(charge);
            t[8] = 0.5 * (p0 * p0 + p1 * p1);
            t[9] = (pa[0] * pa[0] + pa[1] * pa[1] + pa[2] * pa[2]) / (2.0 * g.kappa_g);
            t[10] = fabs(G);
            t[11] = fabs(div);
            t[12] = fabs(charge);
#pragma unroll
            for (int k = 0; k < NQ; ++k) acc[k] = k < kU1Sums ? acc[k] + t[k] : fmax(acc[k], t[k]);
        } else {
            double q0 = p0 + ck * F0, q1 = p1 + ck * F1;
            if (MODE == kU1Kick) {
                q0 += ck2 * F0;
                q1 += ck2 * F1;
            }
            g.pi[0][n] = q0;
            g.pi[1][n] = q1;
            double qa[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                qa[i] = pa[i] + ck * FA[i];
                if (MODE == kU1Kick) qa[i] += ck2 * FA[i];
                g.piA[i][n] = qa[i];
            }
            if (MODE == kU1Kick && g.phi_out[0]) {
                g.phi_out[0][n] = pr;
                g.phi_out[1][n] = pim;
#pragma unroll
                for (int i = 0; i < 3; ++i) g.A_out[i][n] = g.A_in[i][n];
            }
            if (MODE == kU1Step) {
                g.phi_out[0][n] = pr + hdP * q0;
                g.phi_out[1][n] = pim + hdP * q1;
#pragma unroll
                for (int i = 0; i < 3; ++i) g.A_out[i][n] = g.A_in[i][n] + hdA * qa[i];
            }
        }
    }
    }

    if constexpr (MODE == kU1Energy) {
        u1_block_sums(acc, lds_red, &g.partials[(size_t)lid * NQ]);
    }
}

// ---------------------------------------------------------------------------
// Self-consistent expansion of the U(1) model (sec. 5.5.2, the b' equation with
// the gauge energies): one-thread kernels between the lattice passes.  An
// energy pass with ck = 0 leaves the raw volume sums in ScaleRecord::sums[0..4]
// (pi part, gradient, potential, electric, magnetic; the a = 1 forms), from
// which the energies at a are
//   E_K = S0/(V a^6), E_G = S1/(V a^2), E_V = S2/V, E_K^A = S3/(V a^4), E_G^A = S4/(V a^4),
// and the kernel of b is
//   K_a = a^{2 alpha+1}/3 kappa^2 [(alpha-2) E_K + alpha E_G + (alpha-1)(E_K^A + E_G^A) + (alpha+1) E_V].
// The weights of the next pass go to ScaleRecord::w in U1Args::dw order.
// ---------------------------------------------------------------------------
struct U1SelfConst {
    double alpha, kappa2, inv_vol;
};

__device__ inline double u1_kernel_b(double a, const double *S, const U1SelfConst &k)
{
    const double a2 = a * a, a4 = a2 * a2, a6 = a4 * a2;
    const double EK = S[0] * k.inv_vol / a6, EG = S[1] * k.inv_vol / a2, EV = S[2] * k.inv_vol;
    const double EA = S[3] * k.inv_vol / a4 + S[4] * k.inv_vol / a4;
    const double al = k.alpha;
    return pow(a, 2.0 * al + 1.0) / 3.0 * k.kappa2 *
           ((al - 2.0) * EK + al * EG + (al - 1.0) * EA + (al + 1.0) * EV);
}

// weights of a kick at the record's a: {ck, a^{1+alpha}, a^{3+alpha}, a^{alpha-1}, 0, 0, ck2}
__global__ void u1_self_kick_w(ScaleRecord *S, double ck, double ck2, double alpha)
{
    const int l = threadIdx.x;
    const double a = S->a;
    const double p = pow(a, l == 1 ? 1.0 + alpha : (l == 2 ? 3.0 + alpha : alpha - 1.0));
    if (l < 7) S->w[l] = l == 0 ? ck : (l == 6 ? ck2 : (l < 4 ? p : 0.0));
}

// The scale-factor update after a summing pass, in the order
//   b += cB K_a(a, before the kick); b += cA K_a(a, after it); b += cA2 K_a(a, after it)
// (leapfrog, reading A3: cB = cA = h/2, or only cA after a start from synchronised
// momenta; velocity-Verlet, reading R1: cA closes the sub-step behind, cA2 opens the
// one ahead), a' = a + h b, then the weights of the drift {h abar^{alpha-3},
// h abar^{alpha-1}}, abar = (a + a')/2, and of the next kicks c1, c2 at a'.
struct GaugeUpdate {
    int on;
    double cB, cA, cA2, h, c1, c2;
};

// That update by the lanes of one wave, from the sums tot (valid in every lane): a' and
// b, and in lanes 0 .. 6 the weights of the passes to come.
struct GaugeNew {
    double a, b, w;
};
__device__ inline GaugeNew gauge_update(const double *tot, double a, double b, const GaugeUpdate &u,
                                        const U1SelfConst &k, int lane)
{
    const double after[5] = {tot[0], tot[1], tot[2], tot[3], tot[4]};
    const double before[5] = {tot[8], tot[1], tot[2], tot[9], tot[4]};
    if (u.cB != 0.0) b += u.cB * u1_kernel_b(a, before, k);
    if (u.cA != 0.0) b += u.cA * u1_kernel_b(a, after, k);
    if (u.cA2 != 0.0) b += u.cA2 * u1_kernel_b(a, after, k);
    const double a1 = a + u.h * b, am = 0.5 * (a + a1);
    const double ex = lane == 1 ? 1.0 + k.alpha : (lane == 2 ? 3.0 + k.alpha : (lane == 4 ? k.alpha - 3.0 : k.alpha - 1.0));
    const double p = pow(lane < 4 ? a1 : am, ex);
    return GaugeNew{a1, b, lane == 0 ? u.c1 : (lane == 6 ? u.c2 : (lane < 4 ? p : u.h * p))};
}

// The block partials of a summing pass of the gauge models (kU1Sums sums, then
// kU1Maxes maxima per block), combined by one block in a fixed order into the record;
// then the update above, its five powers side by side in the lanes of one wave, and,
// with `host`, a copy of the record in pinned host memory.  One launch of one block
// behind each pass instead of four one-thread kernels (5 us each at any size).
constexpr int kGaugeFinishThreads = 256;
__global__ void __launch_bounds__(kGaugeFinishThreads) gauge_finish(const double *partials, int nb,
                                                                    const ScaleRecord *Sin, ScaleRecord *S,
                                                                    const GaugeUpdate u, const U1SelfConst k,
                                                                    ScaleRecord *host)
{
    constexpr int NQ = kU1Sums + kU1Maxes, NT = kGaugeFinishThreads;
    __shared__ double lds_red[(NT / 64) * NQ];
    __shared__ double tot[NQ];
    const int tid = threadIdx.x;
    double part[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) part[q] = 0.0;
    for (int i = tid; i < nb; i += NT) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const double v = partials[(size_t)i * NQ + q];
            part[q] = q < kU1Sums ? part[q] + v : fmax(part[q], v);
        }
    }
    u1_block_sums(part, lds_red, tot);
    __syncthreads();
    if (tid < kU1Sums) S->sums[tid] = tot[tid];
    else if (tid < NQ) S->maxes[tid - kU1Sums] = tot[tid];
    if (tid >= 64) return;
    if (u.on) {
        const GaugeNew n = gauge_update(tot, Sin->a, Sin->b, u, k, tid);
        if (tid < 7) S->w[tid] = n.w;
        if (tid == 0) {
            S->a = n.a;
            S->b = n.b;
        }
    }
    if (host) {
        __threadfence();   // the wave's stores to the record before its loads of them
        static_assert(sizeof(ScaleRecord) == 32 * sizeof(double), "record size");
        if (tid < 32) ((double *)host)[tid] = load_agent((const double *)S + tid);
    }
}

// A drift that begins with the finish of the summing pass before it, on small lattices:
// every block adds the nb partials itself (in gauge_finish's order), its first wave
// applies the update to the record `in`, and block 0 writes the new record to `out`,
// so a sub-step takes two launches instead of three (U(1) 16^3, ten leapfrog steps with
// their energies 180 -> 160 us; SU(2) 32^3 273 -> 257).
struct GaugeFin {
    const double *partials;
    int nb;
    const ScaleRecord *in;
    ScaleRecord *out;
    GaugeUpdate u;
    U1SelfConst k;
};

// the drift weights h abar^{alpha-3} and h abar^{alpha-1} (blocks of kGaugeFinishThreads)
__device__ inline void gauge_fin_prologue(const GaugeFin &F, double &hd, double &hdA)
{
    constexpr int NQ = kU1Sums, NT = kGaugeFinishThreads;
    __shared__ double lds_red[(NT / 64) * NQ];
    __shared__ double w[7];
    const int tid = threadIdx.x;
    double part[NQ], tot[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) part[q] = 0.0;
    for (int i = tid; i < F.nb; i += NT) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) part[q] += F.partials[(size_t)i * (kU1Sums + kU1Maxes) + q];
    }
    block_sums<NT, NQ>(part, lds_red, tot);
    if (tid < 64) {
        const GaugeNew n = gauge_update(tot, F.in->a, F.in->b, F.u, F.k, tid);
        if (tid < 7) w[tid] = n.w;
        if (blockIdx.x == 0) {
            if (tid < 7) F.out->w[tid] = n.w;
            if (tid == 0) {
                F.out->a = n.a;
                F.out->b = n.b;
            }
        }
    }
    __syncthreads();
    hd = w[4];
    hdA = w[5];
}

// Drift only, with the record's weights hd = dw[4], hdA = dw[5]: phi' = phi + hd pi,
// A_i' = A_i + hdA piA_i, one site per thread.  A site's drift reads nothing else, so
// it runs in place (15 arrays of traffic, no forces, no copy back after the call).
template <bool FIN>
__global__ void __launch_bounds__(kGaugeFinishThreads) u1_drift(const U1Args g, size_t vol, const GaugeFin F)
{
    const size_t n = (size_t)blockIdx.x * kGaugeFinishThreads + threadIdx.x;
    const bool on = n < vol;
    double f[2], p[2], A[3], q[3];   // loaded ahead of the prologue's sums
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        f[c] = on ? g.phi_in[c][n] : 0.0;
        p[c] = on ? g.pi[c][n] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        A[i] = on ? g.A_in[i][n] : 0.0;
        q[i] = on ? g.piA[i][n] : 0.0;
    }
    double hd, hdA;
    if constexpr (FIN) {
        gauge_fin_prologue(F, hd, hdA);
    } else {
        hd = g.dw[4];
        hdA = g.dw[5];
    }
    if (!on) return;
#pragma unroll
    for (int c = 0; c < 2; ++c) g.phi_out[c][n] = f[c] + hd * p[c];
#pragma unroll
    for (int i = 0; i < 3; ++i) g.A_out[i][n] = A[i] + hdA * q[i];
}

// The passes of u1_stage for lattices whose rows fit a block (N up to 512), with
// the transcendental work shared between neighbouring sites.  A block owns TY whole
// x rows, one thread per site (threads rounded up to whole wavefronts), and marches
// z over [z0, z1).  Per plane every site evaluates its own three plaquette sines
// sin theta_ij(n) and its three link phases (cos, sin)(e dx A_i(n)) once; the values
// at n - x and n - y are read from LDS, those at n - z are carried in registers from
// the previous plane, and the row y0 - 1 below the block is evaluated by the block's
// threads, one operation each.  Every angle is formed by the same expression, in the
// same order, as in u1_stage, which evaluates 9 sines and 6 phases per site and reads
// 44 values.  Bound at 128^3 by memory and by what one block of eight wavefronts per CU
// keeps in flight: step pass 62 us over lattices in turn, 357 MB through the L2 misses at
// 5.7 TB/s, waves issuing vector work in 17% of their cycles and waiting in 21% (66 us
// with an LDS array per value, whose addresses took 150 more instructions per plane, and
// in a kernel with the row length known at compile time), energy pass 63 (67).  96^3 step
// pass 30.5 us (32.1; u1_stage 57), energy pass 31 (33; u1_stage 115), kick-and-sums 32.2
// (33.4): the sines, whose vector work takes a quarter of the wave cycles.
constexpr int kU1SpanThreads = 512;
// LDS (doubles): two records of seven values per x position and row, the fields' on the
// rows y0 - 1 .. y0 + TY, the sines' and phases' on y0 - 1 .. y0 + TY - 1.  A site reads its
// neighbours' records at constant offsets from the addresses of five places, formed once
// (an array per value took an address each, a third of the loop's integer instructions);
// seven, an odd number, spreads neighbouring records over the banks.
constexpr int kU1Rec = 7;
enum U1Field : int { kU1Psi = 0, kU1Ax = 4, kU1Az = 5, kU1Ay = 6 };   // psi: two parities of (psi0, psi1)
enum U1Trig : int { kU1Sxy = 0, kU1Syz = 1, kU1Cy = 2, kU1Sy = 3, kU1Sxz = 4, kU1Cx = 5, kU1Sx = 6 };
inline size_t u1_span_lds(int N, int TY) { return (size_t)kU1Rec * N * (2 * (size_t)TY + 3); }

template <int HPT, int MODE>
__global__ void __launch_bounds__(kU1SpanThreads) u1_span(const U1Args g, int TY)
{
    extern __shared__ double u1_lds[];
    constexpr bool EN = MODE == kU1Energy || MODE == kU1KickSums;   // ends with the reduction
    constexpr int NQ = kU1Sums + kU1Maxes;
    __shared__ double lds_red[EN ? (kU1SpanThreads / 64) * NQ : 1];

    const int N = g.N, NT = blockDim.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int chunks = (N + g.zc - 1) / g.zc;
    const int bz = lid % chunks;
    const int by = lid / chunks;
    const int y0 = by * TY, nr = min(TY, N - y0);   // the last block may own fewer rows
    const int z0 = bz * g.zc;
    const int z1 = min(z0 + g.zc, N);
    const bool own = tid < nr * N;            // threads past the rows load and store nothing
    const int r = own ? tid / N + 1 : 1;      // LDS row of this thread's site (rows 0 .. nr + 1 stand for y0 - 1 .. y0 + nr)
    const int x = own ? tid - (r - 1) * N : 0;
    const int xm = x == 0 ? N - 1 : x - 1, xp = x == N - 1 ? 0 : x + 1;

    // LDS places: this site and its neighbours in the field records (f_*) and the sines'
    // (t_*), whose rows 0 .. nr + 1 stand for y0 - 1 .. y0 + nr.  psi is double-buffered by
    // plane parity, so that storing plane z + 1 cannot race with the last reads of plane z;
    // the other values are read before the barrier that the next plane's stores follow.
    double *const F = u1_lds, *const S = F + kU1Rec * (TY + 2) * N;
    const int ro = kU1Rec * (r * N + x), rxm = kU1Rec * (r * N + xm), rdn = ro - kU1Rec * N;
    double *const f_o = F + ro, *const f_dn = F + rdn, *const f_up = F + ro + kU1Rec * N;
    double *const f_xm = F + rxm, *const f_xp = F + kU1Rec * (r * N + xp);
    double *const t_o = S + ro, *const t_dn = S + rdn, *const t_xm = S + rxm;
    double *const top = F + kU1Rec * (nr + 1) * N;   // row nr + 1; its A_y holds A_y(row 0, z + 1)

    const unsigned NN = (unsigned)N * (unsigned)N;   // 8 N^3 < 2^32
    const unsigned so = (unsigned)((y0 + r - 1) * N + x);   // site offset within a plane
    const int yb = (y0 == 0 ? N - 1 : y0 - 1) * N;
    const int yt = ((y0 + nr) % N) * N;
    const int NH = 2 * N, NOP = 3 * N;        // halo cells and halo-row operations per plane
    const int op0 = tid / N, hx0 = tid - op0 * N, dop = NT / N, dhx = NT - dop * N;   // this thread's first, and the step

    const double edx = g.e * g.dx;
    const double inv_dx2 = 1.0 / (g.dx * g.dx);
    const double inv_edx3 = 1.0 / (g.e * g.dx * g.dx * g.dx);
    double ck = g.ck, ck2 = g.ck2, la1 = g.la1, la3 = g.la3, lm1 = g.lam1, hd = g.hd, hdA = g.hdA;
    if (g.dw) {
        ck = g.dw[0];
        la1 = g.dw[1];
        la3 = g.dw[2];
        lm1 = g.dw[3];
        hd = g.dw[4];
        hdA = g.dw[5];
        ck2 = g.dw[6];
    }

    // halo cells: c < N is row 0 (y0 - 1), else row nr + 1 (y0 + nr)
    double *hc[HPT];   // the cell's record
    int hx[HPT];
    unsigned hoff[HPT];
    bool hval[HPT], hbot[HPT];
#pragma unroll
    for (int j = 0; j < HPT; ++j) {
        const int c = tid + j * NT;
        hval[j] = c < NH;
        hbot[j] = c < N;
        hx[j] = hbot[j] ? c : (hval[j] ? c - N : 0);
        hc[j] = (hbot[j] ? F : top) + kU1Rec * hx[j];
        hoff[j] = hval[j] ? (unsigned)((hbot[j] ? yb : yt) + hx[j]) : 0u;
    }

    double wm[2], w0[2], wp[2];   // psi at z - 1, z, z + 1
    double a0[3], a1[3];          // A at z, z + 1
    double czm, szm, sxzm, syzm;  // link phase of A_z and sines theta_xz, theta_yz at n - z
    double hp0[HPT], hp1[HPT], hax[HPT], hay[HPT], haz[HPT], hayn[HPT];
    double acc[NQ];   // energy mode: the site terms of u1_stage, summed over the column
#pragma unroll
    for (int k = 0; k < NQ; ++k) acc[k] = 0.0;

    // ---- prologue: window, A, halo rows of plane z0, carried values of plane z0 - 1
    {
        const unsigned om = (unsigned)(z0 == 0 ? N - 1 : z0 - 1) * NN;
        const unsigned o0 = (unsigned)z0 * NN;
        const unsigned o1 = (unsigned)((z0 + 1) % N) * NN;
        double am[3];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            wm[c] = ld32(g.phi_in[c], om + so);
            w0[c] = ld32(g.phi_in[c], o0 + so);
            wp[c] = ld32(g.phi_in[c], o1 + so);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            am[i] = ld32(g.A_in[i], om + so);
            a0[i] = ld32(g.A_in[i], o0 + so);
            a1[i] = ld32(g.A_in[i], o1 + so);
        }
        if (own) f_o[kU1Az] = am[2];
#pragma unroll
        for (int j = 0; j < HPT; ++j) {
            hp0[j] = hp1[j] = hax[j] = hay[j] = haz[j] = hayn[j] = 0.0;
            if (hval[j]) {
                hp0[j] = ld32(g.phi_in[0], o0 + hoff[j]);
                hp1[j] = ld32(g.phi_in[1], o0 + hoff[j]);
                hax[j] = ld32(g.A_in[0], o0 + hoff[j]);
                haz[j] = ld32(g.A_in[2], o0 + hoff[j]);
                if (hbot[j]) {
                    hay[j] = ld32(g.A_in[1], o0 + hoff[j]);
                    hayn[j] = ld32(g.A_in[1], o1 + hoff[j]);
                } else {
                    hc[j][kU1Az] = ld32(g.A_in[2], om + hoff[j]);
                }
            }
        }
        __syncthreads();
        const double txz = edx * ((f_xp[kU1Az] - am[2]) - a0[0] + am[0]);
        const double tyz = edx * ((f_up[kU1Az] - am[2]) - a0[1] + am[1]);
        sxzm = lat_sin(txz);
        syzm = lat_sin(tyz);
        lat_sincos(edx * am[2], &szm, &czm);
        __syncthreads();
    }

    for (int z = z0; z < z1; ++z) {
        const unsigned oz = (unsigned)z * NN;
        const int q = kU1Psi + 2 * ((z - z0) & 1);   // this plane's psi
        // (A) plane z into LDS
        if (own) {
            f_o[q] = w0[0];
            f_o[q + 1] = w0[1];
            f_o[kU1Ax] = a0[0];
            f_o[kU1Ay] = a0[1];
            f_o[kU1Az] = a0[2];
        }
#pragma unroll
        for (int j = 0; j < HPT; ++j) {
            if (hval[j]) {
                hc[j][q] = hp0[j];
                hc[j][q + 1] = hp1[j];
                hc[j][kU1Ax] = hax[j];
                hc[j][kU1Az] = haz[j];
                if (hbot[j]) {
                    hc[j][kU1Ay] = hay[j];
                    top[kU1Rec * hx[j] + kU1Ay] = hayn[j];
                }
            }
        }
        __syncthreads();

        // (B0) loads for the next plane: psi, A of plane z + 2 and the halo rows
        // of plane z + 1 (indices clamped to valid planes after the chunk's end)
        int z2 = min(z + 2, z1);
        if (z2 >= N) z2 -= N;
        int zh = min(z + 1, z1 - 1);
        if (zh >= N) zh -= N;
        int zhn = zh + 1;
        if (zhn >= N) zhn -= N;
        const unsigned o2 = (unsigned)z2 * NN, oh = (unsigned)zh * NN, ohn = (unsigned)zhn * NN;
        double nps[2], na[3];
#pragma unroll
        for (int c = 0; c < 2; ++c) nps[c] = ld32(g.phi_in[c], o2 + so);
#pragma unroll
        for (int i = 0; i < 3; ++i) na[i] = ld32(g.A_in[i], o2 + so);
#pragma unroll
        for (int j = 0; j < HPT; ++j) {
            if (hval[j]) {
                hp0[j] = ld32(g.phi_in[0], oh + hoff[j]);
                hp1[j] = ld32(g.phi_in[1], oh + hoff[j]);
                hax[j] = ld32(g.A_in[0], oh + hoff[j]);
                haz[j] = ld32(g.A_in[2], oh + hoff[j]);
                if (hbot[j]) {
                    hay[j] = ld32(g.A_in[1], oh + hoff[j]);
                    hayn[j] = ld32(g.A_in[1], ohn + hoff[j]);
                }
            }
        }

        // (B) own plaquette sines and link phases into LDS; then the halo
        // row's, one operation per thread
        double th[3];   // own plaquette angles (the energy mode's magnetic term)
        double ss[3], ps[3], pc[3];   // their sines; sine and cosine of the link phases
        {
            const double txy = edx * ((f_xp[kU1Ay] - a0[1]) - f_up[kU1Ax] + a0[0]);
            const double txz = edx * ((f_xp[kU1Az] - a0[2]) - a1[0] + a0[0]);
            const double tyz = edx * ((f_up[kU1Az] - a0[2]) - a1[1] + a0[1]);
            th[0] = txy;
            th[1] = txz;
            th[2] = tyz;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double t = j == 0 ? txy : (j == 1 ? txz : tyz);
                ss[j] = lat_sin(t);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) lat_sincos(edx * a0[j], &ps[j], &pc[j]);
            if (own) {
                t_o[kU1Sxy] = ss[0];
                t_o[kU1Sxz] = ss[1];
                t_o[kU1Syz] = ss[2];
                t_o[kU1Sx] = ps[0];
                t_o[kU1Cx] = pc[0];
                t_o[kU1Sy] = ps[1];
                t_o[kU1Cy] = pc[1];
            }
        }
        for (int id = tid, op = op0, hxo = hx0; id < NOP; id += NT) {
            double *const f = F + kU1Rec * hxo, *const t = S + kU1Rec * hxo;
            if (op == 0) {
                double sv, cv;
                lat_sincos(edx * f[kU1Ay], &sv, &cv);
                t[kU1Sy] = sv;
                t[kU1Cy] = cv;
            } else if (op == 1) {
                const double ayp = hxo == N - 1 ? F[kU1Ay] : f[kU1Rec + kU1Ay];
                t[kU1Sxy] = lat_sin(edx * ((ayp - f[kU1Ay]) - f[kU1Rec * N + kU1Ax] + f[kU1Ax]));
            } else {
                t[kU1Syz] = lat_sin(edx * ((f[kU1Rec * N + kU1Az] - f[kU1Az]) - top[kU1Rec * hxo + kU1Ay] + f[kU1Ay]));
            }
            op += dop;
            hxo += dhx;
            if (hxo >= N) {
                hxo -= N;
                ++op;
            }
        }
        __syncthreads();

        // (C) forces, kick, drift
        if (own) {
            const unsigned o = oz + so;
            double pq[2], pa[3];
#pragma unroll
            for (int c = 0; c < 2; ++c) pq[c] = ld32(g.pi[c], o);
#pragma unroll
            for (int i = 0; i < 3; ++i) pa[i] = ld32(g.piA[i], o);
            const double sxy = ss[0], sxz = ss[1], syz = ss[2];
            const double mag[3] = {(sxy - t_dn[kU1Sxy]) + (sxz - sxzm),
                                   (-sxy + t_xm[kU1Sxy]) + (syz - syzm),
                                   (-sxz + t_xm[kU1Sxz]) + (-syz + t_dn[kU1Syz])};
            const double pr = w0[0], pim = w0[1];
            double d2r = 0.0, d2i = 0.0, J[3], grad2 = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                double qr, qi, rr, ri, sm, cm;
                if (i == 0) {
                    qr = f_xp[q]; qi = f_xp[q + 1];
                    rr = f_xm[q]; ri = f_xm[q + 1];
                    sm = t_xm[kU1Sx]; cm = t_xm[kU1Cx];
                } else if (i == 1) {
                    qr = f_up[q]; qi = f_up[q + 1];
                    rr = f_dn[q]; ri = f_dn[q + 1];
                    sm = t_dn[kU1Sy]; cm = t_dn[kU1Cy];
                } else {
                    qr = wp[0]; qi = wp[1];
                    rr = wm[0]; ri = wm[1];
                    sm = szm; cm = czm;
                }
                const double s = -ps[i], c = pc[i];   // V_i(n) = c + i s
                const double ar = c * qr - s * qi, ai = c * qi + s * qr;
                const double br = cm * rr - sm * ri, bi = cm * ri + sm * rr;
                d2r += ar - 2.0 * pr + br;
                d2i += ai - 2.0 * pim + bi;
                J[i] = g.e / g.dx * (pr * ai - pim * ar);
                if constexpr (EN) {
                    const double dr = ar - pr, di = ai - pim;
                    grad2 += dr * dr + di * di;
                }
            }
            const double m2 = 0.5 * (pr * pr + pim * pim);
            const double vp = 0.5 * g.lam * (m2 - g.v * g.v);
            const double F0 = la1 * (d2r * inv_dx2) - la3 * (vp * pr);
            const double F1 = la1 * (d2i * inv_dx2) - la3 * (vp * pim);
            const double q0 = pq[0] + ck * F0, q1 = pq[1] + ck * F1;
            if constexpr (MODE == kU1Energy) {
                // the energies and Gauss terms of u1_stage's energy mode
                double t[NQ];
                t[0] = 0.5 * (q0 * q0 + q1 * q1);
                t[1] = grad2 * inv_dx2 * 0.5;
                const double u = m2 - g.v * g.v;
                t[2] = 0.25 * g.lam * u * u;
                double ka = 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const double FA = la1 * (g.kappa_g * J[i]) - lm1 * (mag[i] * inv_edx3);
                    const double sa = pa[i] + ck * FA;
                    ka += sa * sa;
                }
                t[3] = ka / (2.0 * g.kappa_g);
                const double hxy = lat_sin(0.5 * th[0]), hxz = lat_sin(0.5 * th[1]), hyz = lat_sin(0.5 * th[2]);
                const double mg = 2.0 * hxy * hxy + 2.0 * hxz * hxz + 2.0 * hyz * hyz;
                t[4] = mg / (g.kappa_g * g.e * g.e * g.dx * g.dx * g.dx * g.dx);
                const int yy = y0 + r - 1;
                const unsigned oxm = oz + (unsigned)(yy * N + xm);
                const unsigned oym = oz + (unsigned)((yy == 0 ? N - 1 : yy - 1) * N + x);
                const unsigned ozm = (unsigned)(z == 0 ? N - 1 : z - 1) * NN + so;
                const double div = ((pa[0] - ld32(g.piA[0], oxm)) + (pa[1] - ld32(g.piA[1], oym)) +
                                    (pa[2] - ld32(g.piA[2], ozm))) / g.dx;
                const double charge = g.e * g.kappa_g * (pr * pq[1] - pim * pq[0]);
                const double G = div - charge;
                t[5] = fabs(G);
                t[6] = fabs(div + charge);
                t[7] = fabs(div) + fabs(charge);
                t[8] = 0.5 * (pq[0] * pq[0] + pq[1] * pq[1]);
                t[9] = (pa[0] * pa[0] + pa[1] * pa[1] + pa[2] * pa[2]) / (2.0 * g.kappa_g);
                t[10] = fabs(G);
                t[11] = fabs(div);
                t[12] = fabs(charge);
#pragma unroll
                for (int k = 0; k < NQ; ++k) acc[k] = k < kU1Sums ? acc[k] + t[k] : fmax(acc[k], t[k]);
            } else {
                constexpr bool two = MODE == kU1KickSums;   // a second kick after the sums
                st32(g.pi[0], o, two ? q0 + ck2 * F0 : q0);
                st32(g.pi[1], o, two ? q1 + ck2 * F1 : q1);
                const bool carry = MODE == kU1Kick && g.phi_out[0];
                if constexpr (MODE == kU1Step) {
                    st32(g.phi_out[0], o, pr + hd * q0);
                    st32(g.phi_out[1], o, pim + hd * q1);
                } else if (carry) {
                    st32(g.phi_out[0], o, pr);
                    st32(g.phi_out[1], o, pim);
                }
                double ka = 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const double FA = la1 * (g.kappa_g * J[i]) - lm1 * (mag[i] * inv_edx3);
                    const double qa = pa[i] + ck * FA;
                    st32(g.piA[i], o, two ? qa + ck2 * FA : qa);
                    if constexpr (MODE == kU1Step) st32(g.A_out[i], o, a0[i] + hdA * qa);
                    else if (carry) st32(g.A_out[i], o, a0[i]);
                    if constexpr (MODE == kU1KickSums) ka += qa * qa;
                }
                if constexpr (MODE == kU1KickSums) {
                    double t[NQ];
                    t[0] = 0.5 * (q0 * q0 + q1 * q1);
                    t[1] = grad2 * inv_dx2 * 0.5;
                    const double u = m2 - g.v * g.v;
                    t[2] = 0.25 * g.lam * u * u;
                    t[3] = ka / (2.0 * g.kappa_g);
                    const double hxy = lat_sin(0.5 * th[0]), hxz = lat_sin(0.5 * th[1]), hyz = lat_sin(0.5 * th[2]);
                    const double mg = 2.0 * hxy * hxy + 2.0 * hxz * hxz + 2.0 * hyz * hyz;
                    t[4] = mg / (g.kappa_g * g.e * g.e * g.dx * g.dx * g.dx * g.dx);
                    t[8] = 0.5 * (pq[0] * pq[0] + pq[1] * pq[1]);
                    t[9] = (pa[0] * pa[0] + pa[1] * pa[1] + pa[2] * pa[2]) / (2.0 * g.kappa_g);
#pragma unroll
                    for (int k = 0; k < kU1Sums; ++k)
                        if (k < 5 || k > 7) acc[k] += t[k];
                }
            }
            czm = pc[2];
            szm = ps[2];
            sxzm = sxz;
            syzm = syz;
        }
        // no barrier here: plane z + 1 goes to the other psi / A buffers, and the
        // sines and phases read above are rewritten only after the next barrier
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            wm[c] = w0[c];
            w0[c] = wp[c];
            wp[c] = nps[c];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            a0[i] = a1[i];
            a1[i] = na[i];
        }
    }

    if constexpr (EN) {
        u1_block_sums(acc, lds_red, &g.partials[(size_t)lid * NQ]);
    }
}

}  // namespace lat
