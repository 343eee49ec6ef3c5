// stage_su2.hpp -- SU(2) doublet with SU(2) links: the leapfrog pass
// (kick of the doublet momenta and electric fields, drift of the doublet and
// the links), the sync half kick, and the energy / Gauss reduction pass.
//
// Lattice system (sec. 3.2 SU(N) toolkit; sec. 5, eqs. higgsSU2-eom, SU2eom,
// GaussSU2-eom, energy-contrib, program variables with f_* = omega_*):
//   doublet Phi = (psi0, psi1)/sqrt2, psi0 = phi0 + i phi1, psi1 = phi2 + i phi3;
//   link U_i(n) = exp(-i g dx B_i^a T_a), T_a = sigma_a/2, stored as the unit
//   quaternion (w, x, y, z) with U = w I - i (x, y, z).sigma;
//   electric field E_i^a(n), conjugate to U_i(n) under U -> exp(-i eps g dx T_a) U.
// Hamiltonian per site: sum_c pi_c^2/2 + sum_i |U_i psi(n+i) - psi|^2/(2 dx^2)
//   + lambda/4 (|Phi|^2 - v^2)^2 + |E|^2/2 + 2/(g^2 dx^4) sum_{i<j} (2 - Tr P_ij),
//   P_ij(n) = U_i(n) U_j(n+i) U_i(n+j)^dag U_j(n)^dag.
// Kicks are minus its derivative:
//   pi_c  += ck [ (D^2 psi)_c - lambda/2 (|Phi|^2 - v^2) phi_c ]
//   E_i^a += ck [ (g/dx) Im(psi^dag T_a U_i psi(n+i))
//                 - 2/(g dx^3) vec_a(U_i sum_{j != i} (S+_ij + S-_ij)) ]
//   S+_ij = U_j(n+i) U_i(n+j)^dag U_j(n)^dag,  S-_ij = U_j(n+i-j)^dag U_i(n-j)^dag U_j(n-j)
// and the drifts phi += hd pi, U <- exp(-i hd g dx E^a T_a) U.
// One thread per site of each plane of a z column; neighbours through the
// caches.  Momenta are read at their own site only and updated in place;
// doublet and links are written out of place (the stencil reads the old values).
#pragma once
#include "common.hpp"
#include "stage_u1.hpp"

namespace lat {

struct SU2Args {
    const double *phi_in[4];
    double *phi_out[4];
    double *pi[4];
    const double *U_in[12];   // link i, component k at 4 i + k
    double *U_out[12];
    double *E[9];             // link i, colour a at 3 i + a
    // kSU2StepAoS: the doublet and the links as one 32-byte record per site
    // (phi0..phi3; w, x, y, z), read from *_in4 and written to *_out4;
    // kSU2StepOut: read from *_in4 and written to the plain arrays
    const double4 *phi_in4;
    double4 *phi_out4;
    const double4 *U_in4[3];
    double4 *U_out4[3];
    int N, tx, ty, tiles_x, tiles_y, zc;   // tile of tx x ty <= 256 sites, z planes per block
    int band;                      // > 0: tiles of a plane per XCD, see su2_stage
    int down;                      // march the z column downward (sites are independent)
    double dx, g, lam, v;
    double ck;   // kick weight
    double hd;   // drift weight of the doublet (time times a^{alpha-3})
    // expanding background (sec. 5.5.2 kernels): the covariant Laplacian and
    // the current scale with la1 = a^{1+alpha}, the potential force with
    // la3 = a^{3+alpha}, the staple force with lam1 = a^{alpha-1}; hdU is the
    // link drift weight (time times a^{alpha-1}).  All 1 (hdU = hd) at a = 1.
    double la1, la3, lam1, hdU;
    // if not null: {ck, la1, la3, lam1, hd, hdU, ck2} from device memory (written by
    // the self-consistent scale-factor update)
    const double *dw;
    double *partials;
    double ck2;  // a second kick weight, applied after the first (and after the sums of kSU2KickSums)
};

// kSU2Drift: the drift alone (su2_drift).
// kSU2KickSums: kicks by ck, forms the volume sums [0, 5) of that state and the momentum
// sums [8, 10) before the kick, then kicks by ck2 (in the energy pass's launch shape;
// Gauss terms not measured: the rest stays zero).  kSU2Kick with output arrays also
// carries the doublet and the links over to them.
enum SU2Mode : int { kSU2Step = 0, kSU2Kick = 1, kSU2Energy = 2, kSU2StepAoS = 3, kSU2Drift = 4, kSU2KickSums = 5,
                     kSU2StepOut = 6 };

// one 32-byte record through a 32-bit byte offset (valid while 32 N^3 < 2^32)
__device__ __forceinline__ double4 ld4(const double4 *base, unsigned i)
{
    return *(const double4 *)((const char *)base + (size_t)(i * 32u));
}
__device__ __forceinline__ void st4(double4 *base, unsigned i, double4 v)
{
    *(double4 *)((char *)base + (size_t)(i * 32u)) = v;
}

// Streamed accesses of the pass (the momenta, read and written once, and the
// output records): non-temporal when NT, so they do not displace the input
// records that neighbouring sites read again from L2.
typedef double su2_nd4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ double ld_s(const double *base, unsigned i)
{
    const double *p = (const double *)((const char *)base + (size_t)(i * 8u));
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT>
__device__ __forceinline__ void st_s(double *base, unsigned i, double v)
{
    double *p = (double *)((char *)base + (size_t)(i * 8u));
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <bool NT>
__device__ __forceinline__ void st4_s(double4 *base, unsigned i, double4 v)
{
    if constexpr (NT) {
        const su2_nd4 w = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(w, (su2_nd4 *)((char *)base + (size_t)(i * 32u)));
    } else {
        st4(base, i, v);
    }
}
constexpr int kSU2Sums = kU1Sums, kSU2Maxes = kU1Maxes;   // the U(1) passes' slots

// unit quaternion q = (w, v) for the matrix w I - i v.sigma
struct Q4 {
    double w, x, y, z;
};

__device__ __forceinline__ Q4 qmul(const Q4 &a, const Q4 &b)
{
    // (a0 - i a.s)(b0 - i b.s) = (a0 b0 - a.b) - i (a0 b + b0 a + a x b).s
    Q4 c;
    c.w = a.w * b.w - (a.x * b.x + a.y * b.y + a.z * b.z);
    c.x = a.w * b.x + b.w * a.x + (a.y * b.z - a.z * b.y);
    c.y = a.w * b.y + b.w * a.y + (a.z * b.x - a.x * b.z);
    c.z = a.w * b.z + b.w * a.z + (a.x * b.y - a.y * b.x);
    return c;
}

__device__ __forceinline__ Q4 qdag(const Q4 &a) { return Q4{a.w, -a.x, -a.y, -a.z}; }

__device__ __forceinline__ Q4 qadd(const Q4 &a, const Q4 &b) { return Q4{a.w + b.w, a.x + b.x, a.y + b.y, a.z + b.z}; }

// exp(-i hgdx e.T) = cos(th/2) - i sin(th/2) e.sigma/|e|, th = hgdx |e|.  Up to
// th/2 = pi/4 both factors come from the polynomials of trig.hpp in (th/2)^2
// (sin(t)/t is the sine polynomial with t = 1 outside), so the usual small angles
// need no square root, no division and no range reduction.
__device__ __forceinline__ Q4 su2_exp(double hgdx, double ex, double ey, double ez)
{
    const double hh = 0.5 * hgdx, e2 = ex * ex + ey * ey + ez * ez, z = hh * hh * e2;
    double f, w;
    if (z <= kQuarterPi * kQuarterPi) {
        f = hh * trig::sin_poly(1.0, z);
        w = trig::cos_poly(z);
    } else {
        const double len = sqrt(e2);
        const trig::SinCos sc = trig::sincos_full(hh * len);
        f = sc.s / len;
        w = sc.c;
    }
    return Q4{w, f * ex, f * ey, f * ez};
}

// (r0 + i s0, r1 + i s1) = U (a + i b, c + i d), U = w I - i v.sigma
__device__ __forceinline__ void qapply(const Q4 &u, double a, double b, double c, double d, double &r0, double &s0,
                                       double &r1, double &s1)
{
    r0 = u.w * a + u.z * b - u.y * c + u.x * d;
    s0 = u.w * b - u.z * a - u.y * d - u.x * c;
    r1 = u.x * b + u.y * a + u.w * c - u.z * d;
    s1 = -u.x * a + u.y * b + u.w * d + u.z * c;
}

// Im(psi^dag T_a chi), a = 1..3, psi = (a + i b, c + i d), chi = (p + i q, r + i s)
__device__ __forceinline__ void isospin(double a, double b, double c, double d, double p, double q, double r, double s,
                                        double &j1, double &j2, double &j3)
{
    j1 = 0.5 * ((a * s - b * r) + (c * q - d * p));
    j2 = 0.5 * ((c * p + d * q) - (a * r + b * s));
    j3 = 0.5 * ((a * q - b * p) - (c * s - d * r));
}

// One site's pass.  Site indices are 32-bit element offsets (the caller
// checks 8 N^3 < 2^32), so every array access is a uniform base plus one
// 32-bit offset.  c[] = (x, y, z), cp[] / cm[] their periodic successors and
// predecessors.
// the pass weights of SU2Args, from device memory if SU2Args::dw is set
struct SU2W {
    double ck, la1, la3, lm1, hd, hdU, ck2;
};

__device__ inline SU2W su2_weights(const SU2Args &g)
{
    if (g.dw) return SU2W{g.dw[0], g.dw[1], g.dw[2], g.dw[3], g.dw[4], g.dw[5], g.dw[6]};
    return SU2W{g.ck, g.la1, g.la3, g.lam1, g.hd, g.hdU, g.ck2};
}

template <int MODE, int NQ, bool NT>
__device__ __forceinline__ void su2_site(const SU2Args &g, const SU2W &wt, const int (&c)[3], const int (&cp)[3],
                                         const int (&cm)[3], double (&acc)[NQ])
{
    const unsigned N = (unsigned)g.N;
    auto off = [&](int x, int y, int z) { return (unsigned)x + N * ((unsigned)y + N * (unsigned)z); };
    // site index with coordinate i replaced by v (and optionally j by u)
    auto at1 = [&](int i, int v) {
        int q[3] = {c[0], c[1], c[2]};
        q[i] = v;
        return off(q[0], q[1], q[2]);
    };
    auto at2 = [&](int i, int v, int j, int u) {
        int q[3] = {c[0], c[1], c[2]};
        q[i] = v;
        q[j] = u;
        return off(q[0], q[1], q[2]);
    };
    constexpr bool AOS = MODE == kSU2StepAoS || MODE == kSU2StepOut, AOS_OUT = MODE == kSU2StepAoS;
    auto L = [&](int i, unsigned m) {
        if constexpr (AOS) {
            const double4 v = ld4(g.U_in4[i], m);
            return Q4{v.x, v.y, v.z, v.w};
        } else {
            return Q4{ld32(g.U_in[4 * i], m), ld32(g.U_in[4 * i + 1], m), ld32(g.U_in[4 * i + 2], m),
                      ld32(g.U_in[4 * i + 3], m)};
        }
    };
    // the doublet at site m as (phi0, phi1, phi2, phi3)
    auto D = [&](unsigned m) {
        if constexpr (AOS) {
            return ld4(g.phi_in4, m);
        } else {
            return double4{ld32(g.phi_in[0], m), ld32(g.phi_in[1], m), ld32(g.phi_in[2], m), ld32(g.phi_in[3], m)};
        }
    };
    const unsigned n = off(c[0], c[1], c[2]);
    const double4 own = D(n);
    const double a0 = own.x, b0 = own.y, c0 = own.z, d0 = own.w;
    const double inv_dx2 = 1.0 / (g.dx * g.dx);
    const double gdx = g.g / g.dx;
    const double mcoef = 2.0 / (g.g * g.dx * g.dx * g.dx);

    double l0 = 0.0, l1 = 0.0, l2 = 0.0, l3 = 0.0;   // sum_i U psi(n+i) - 2 psi + U^dag psi(n-i)
    double grad2 = 0.0;
    double FE[9];
    Q4 Ul[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) Ul[i] = L(i, n);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const unsigned np = at1(i, cp[i]), nm = at1(i, cm[i]);
        double r0, s0, r1, s1;
        const double4 dp = D(np), dm = D(nm);
        qapply(Ul[i], dp.x, dp.y, dp.z, dp.w, r0, s0, r1, s1);
        double t0, u0, t1, u1;
        qapply(qdag(L(i, nm)), dm.x, dm.y, dm.z, dm.w, t0, u0, t1, u1);
        l0 += r0 - 2.0 * a0 + t0;
        l1 += s0 - 2.0 * b0 + u0;
        l2 += r1 - 2.0 * c0 + t1;
        l3 += s1 - 2.0 * d0 + u1;
        if (MODE == kSU2Energy || MODE == kSU2KickSums) {
            const double e0 = r0 - a0, e1 = s0 - b0, e2 = r1 - c0, e3 = s1 - d0;
            grad2 += e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
        }
        double j1, j2, j3;
        isospin(a0, b0, c0, d0, r0, s0, r1, s1, j1, j2, j3);
        // staple sum of link i
        Q4 S{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (j == i) continue;
            const Q4 Sp = qmul(qmul(L(j, np), qdag(L(i, at1(j, cp[j])))), qdag(Ul[j]));   // U_j(n+i) U_i(n+j)^dag U_j^dag
            const Q4 Sm = qmul(qmul(qdag(L(j, at2(i, cp[i], j, cm[j]))), qdag(L(i, at1(j, cm[j])))),
                               L(j, at1(j, cm[j])));   // U_j(n+i-j)^dag U_i(n-j)^dag U_j(n-j)
            S = qadd(S, qadd(Sp, Sm));
        }
        const Q4 W = qmul(Ul[i], S);
        FE[3 * i + 0] = wt.la1 * (gdx * j1) - wt.lm1 * (mcoef * W.x);
        FE[3 * i + 1] = wt.la1 * (gdx * j2) - wt.lm1 * (mcoef * W.y);
        FE[3 * i + 2] = wt.la1 * (gdx * j3) - wt.lm1 * (mcoef * W.z);
    }
    const double m2 = 0.5 * (a0 * a0 + b0 * b0 + c0 * c0 + d0 * d0);
    const double vp = 0.5 * g.lam * (m2 - g.v * g.v);
    const double F[4] = {wt.la1 * (l0 * inv_dx2) - wt.la3 * (vp * a0), wt.la1 * (l1 * inv_dx2) - wt.la3 * (vp * b0),
                         wt.la1 * (l2 * inv_dx2) - wt.la3 * (vp * c0), wt.la1 * (l3 * inv_dx2) - wt.la3 * (vp * d0)};
    double pv[4], ev[9];
#pragma unroll
    for (int k = 0; k < 4; ++k) pv[k] = ld_s<NT>((const double *)g.pi[k], n);
#pragma unroll
    for (int k = 0; k < 9; ++k) ev[k] = ld_s<NT>((const double *)g.E[k], n);

    if (MODE == kSU2Energy) {
        double kin = 0.0, ke = 0.0, kin0 = 0.0, ke0 = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double s = pv[k] + wt.ck * F[k];
            kin += s * s;
            kin0 += pv[k] * pv[k];
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const double s = ev[k] + wt.ck * FE[k];
            ke += s * s;
            ke0 += ev[k] * ev[k];
        }
        acc[8] += 0.5 * kin0;
        acc[9] += 0.5 * ke0;
        acc[0] += 0.5 * kin;
        acc[1] += grad2 * inv_dx2 * 0.5;
        const double u = m2 - g.v * g.v;
        acc[2] += 0.25 * g.lam * u * u;
        acc[3] += 0.5 * ke;
        // magnetic: 2 - Tr P = 2 |p|^2 / (1 + p0) per plaquette (unitary P)
        double mg = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i + 1; j < 3; ++j) {
                const Q4 Pij = qmul(qmul(Ul[i], L(j, at1(i, cp[i]))), qmul(qdag(L(i, at1(j, cp[j]))), qdag(Ul[j])));
                mg += 2.0 * (Pij.x * Pij.x + Pij.y * Pij.y + Pij.z * Pij.z) / (1.0 + Pij.w);
            }
        acc[4] += 2.0 * mg / (g.g * g.g * g.dx * g.dx * g.dx * g.dx);
        // Gauss residual of the stored pairing: covariant backward divergence
        // of E (E_i(n-i) carried to n by U_i(n-i)^dag (E.sigma) U_i(n-i), a
        // rotation of the vector by the inverse of U's) minus the charge
        double dv[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const unsigned nm = at1(i, cm[i]);
            const Q4 u = L(i, nm);
            const double ex = ld32((const double *)g.E[3 * i], nm), ey = ld32((const double *)g.E[3 * i + 1], nm),
                         ez = ld32((const double *)g.E[3 * i + 2], nm);
            // t = 2 v x e ; e' = e - w t + v x t  (rotation by the inverse)
            const double tx2 = 2.0 * (u.y * ez - u.z * ey), ty2 = 2.0 * (u.z * ex - u.x * ez),
                         tz2 = 2.0 * (u.x * ey - u.y * ex);
            const double rx = ex - u.w * tx2 + (u.y * tz2 - u.z * ty2);
            const double ry = ey - u.w * ty2 + (u.z * tx2 - u.x * tz2);
            const double rz = ez - u.w * tz2 + (u.x * ty2 - u.y * tx2);
            dv[0] += (ev[3 * i] - rx) / g.dx;
            dv[1] += (ev[3 * i + 1] - ry) / g.dx;
            dv[2] += (ev[3 * i + 2] - rz) / g.dx;
        }
        double q1, q2, q3;
        isospin(a0, b0, c0, d0, pv[0], pv[1], pv[2], pv[3], q1, q2, q3);
        const double ch[3] = {g.g * q1, g.g * q2, g.g * q3};
        double G2 = 0.0, D2 = 0.0, C2 = 0.0, S2 = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            G2 += (dv[k] - ch[k]) * (dv[k] - ch[k]);
            D2 += dv[k] * dv[k];
            C2 += ch[k] * ch[k];
            S2 += (dv[k] + ch[k]) * (dv[k] + ch[k]);
        }
        const double Gn = sqrt(G2), Dn = sqrt(D2), Cn = sqrt(C2);
        acc[5] += Gn;
        acc[6] += sqrt(S2);
        acc[7] += Dn + Cn;
        acc[10] = fmax(acc[10], Gn);
        acc[11] = fmax(acc[11], Dn);
        acc[12] = fmax(acc[12], Cn);
    } else {
        double pn[4], en[9];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pn[k] = pv[k] + wt.ck * F[k];
            st_s<NT>(g.pi[k], n, MODE == kSU2KickSums ? pn[k] + wt.ck2 * F[k] : pn[k]);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            en[k] = ev[k] + wt.ck * FE[k];
            st_s<NT>(g.E[k], n, MODE == kSU2KickSums ? en[k] + wt.ck2 * FE[k] : en[k]);
        }
        if constexpr (MODE == kSU2KickSums) {
            double kin = 0.0, ke = 0.0, kin0 = 0.0, ke0 = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                kin += pn[k] * pn[k];
                kin0 += pv[k] * pv[k];
            }
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                ke += en[k] * en[k];
                ke0 += ev[k] * ev[k];
            }
            acc[8] += 0.5 * kin0;
            acc[9] += 0.5 * ke0;
            acc[0] += 0.5 * kin;
            acc[1] += grad2 * inv_dx2 * 0.5;
            const double u = m2 - g.v * g.v;
            acc[2] += 0.25 * g.lam * u * u;
            acc[3] += 0.5 * ke;
            double mg = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = i + 1; j < 3; ++j) {
                    const Q4 Pij =
                        qmul(qmul(Ul[i], L(j, at1(i, cp[i]))), qmul(qdag(L(i, at1(j, cp[j]))), qdag(Ul[j])));
                    mg += 2.0 * (Pij.x * Pij.x + Pij.y * Pij.y + Pij.z * Pij.z) / (1.0 + Pij.w);
                }
            acc[4] += 2.0 * mg / (g.g * g.g * g.dx * g.dx * g.dx * g.dx);
        }
        if (MODE == kSU2Kick && g.phi_out[0]) {
            st32(g.phi_out[0], n, a0);
            st32(g.phi_out[1], n, b0);
            st32(g.phi_out[2], n, c0);
            st32(g.phi_out[3], n, d0);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                st32(g.U_out[4 * i], n, Ul[i].w);
                st32(g.U_out[4 * i + 1], n, Ul[i].x);
                st32(g.U_out[4 * i + 2], n, Ul[i].y);
                st32(g.U_out[4 * i + 3], n, Ul[i].z);
            }
        }
        if (MODE == kSU2Step || AOS) {
            const double4 po{a0 + wt.hd * pn[0], b0 + wt.hd * pn[1], c0 + wt.hd * pn[2], d0 + wt.hd * pn[3]};
            if constexpr (AOS_OUT) {
                st4_s<NT>(g.phi_out4, n, po);
            } else {
                st_s<NT>(g.phi_out[0], n, po.x);
                st_s<NT>(g.phi_out[1], n, po.y);
                st_s<NT>(g.phi_out[2], n, po.z);
                st_s<NT>(g.phi_out[3], n, po.w);
            }
            const double hgdx = wt.hdU * g.g * g.dx;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const Q4 R = su2_exp(hgdx, en[3 * i], en[3 * i + 1], en[3 * i + 2]);
                const Q4 Un = qmul(R, Ul[i]);
                if constexpr (AOS_OUT) {
                    st4_s<NT>(g.U_out4[i], n, double4{Un.w, Un.x, Un.y, Un.z});
                } else {
                    st_s<NT>(g.U_out[4 * i], n, Un.w);
                    st_s<NT>(g.U_out[4 * i + 1], n, Un.x);
                    st_s<NT>(g.U_out[4 * i + 2], n, Un.y);
                    st_s<NT>(g.U_out[4 * i + 3], n, Un.z);
                }
            }
        }
    }
}

// Drift only, with the record's weights hd = dw[4], hdU = dw[5], on the plain
// arrays, one site per thread and in place (a site's drift reads nothing else): the
// doublet phi + hd pi and the links exp(-i hdU g dx E.T) U, the step pass's drift
// formed by the same expressions.  Reads 29 arrays and writes 16, with no forces.
template <bool FIN>
__global__ void __launch_bounds__(kGaugeFinishThreads) su2_drift(const SU2Args g, unsigned vol, const GaugeFin F)
{
    const unsigned n = blockIdx.x * (unsigned)kGaugeFinishThreads + threadIdx.x;
    double hd, hdU;
    if constexpr (FIN) {
        gauge_fin_prologue(F, hd, hdU);
    } else {
        hd = g.dw[4];
        hdU = g.dw[5];
    }
    if (n >= vol) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) g.phi_out[k][n] = g.phi_in[k][n] + hd * g.pi[k][n];
    const double hgdx = hdU * g.g * g.dx;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double ex = g.E[3 * i][n], ey = g.E[3 * i + 1][n], ez = g.E[3 * i + 2][n];
        const Q4 R = su2_exp(hgdx, ex, ey, ez);
        const Q4 U{g.U_in[4 * i][n], g.U_in[4 * i + 1][n], g.U_in[4 * i + 2][n], g.U_in[4 * i + 3][n]};
        const Q4 Un = qmul(R, U);
        g.U_out[4 * i][n] = Un.w;
        g.U_out[4 * i + 1][n] = Un.x;
        g.U_out[4 * i + 2][n] = Un.y;
        g.U_out[4 * i + 3][n] = Un.z;
    }
}

// Block = tx x ty sites (at most 256, tx and ty at run time so that any N is cut with
// few idle threads) of a z column [z0, z0 + zc).  Plane-wide order (band = 0): logical
// blocks are dealt to the XCDs in contiguous ranges, x tile fastest, then y tile, then
// z chunk, so an XCD's resident blocks march whole planes together.  Band order
// (band > 0): XCD k owns the tiles [k band, (k + 1) band) of a plane over all z chunks
// (in reverse when marching down; band = tiles / 8 rounded up, the last XCD's may be
// missing), so its resident blocks cover a compact region and the records of the
// planes z - 1, z, z + 1 that a site's stencil reads stay in that XCD's L2 between
// their uses.
// Two waves per SIMD in every mode: the kick-only and energy passes then
// spill 24 and 28 bytes per lane to scratch instead of holding 256 VGPRs and
// 6 AGPRs at one wave (energy pass 361 -> 298 us at 128^3, self-consistent
// leapfrog step 1316 -> 1133 us); the record step pass fits in 240 VGPRs.
constexpr int kSU2Threads = 256;
template <int MODE, bool STREAM>
__global__ void __launch_bounds__(kSU2Threads) __attribute__((amdgpu_waves_per_eu(2))) su2_stage(const SU2Args g)
{
    constexpr int NT = kSU2Threads;
    constexpr int NQ = kSU2Sums + kSU2Maxes;
    __shared__ double lds_red[(NT / 64) * NQ];

    const int tid = threadIdx.x;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int N = g.N, tiles = g.tiles_x * g.tiles_y;
    int t, bz;
    if (g.band > 0) {
        const int per = gridDim.x / 8;   // the host launches 8 band z-chunk blocks
        const int xcd = lid / per, r = lid % per;
        t = xcd * g.band + r % g.band;
        bz = r / g.band;
        if (g.down) bz = (N + g.zc - 1) / g.zc - 1 - bz;
    } else {
        t = lid % tiles;
        bz = lid / tiles;
    }
    const int iy = tid / g.tx, ix = tid - iy * g.tx;
    const bool on = t < tiles && iy < g.ty;
    const int x = (t % g.tiles_x) * g.tx + ix, y = (t / g.tiles_x) * g.ty + iy;
    const int z0 = bz * g.zc, z1 = min(z0 + g.zc, N);

    double acc[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) acc[k] = 0.0;

    const SU2W wt = su2_weights(g);
    if (on && x < N && y < N) {
        int c[3] = {x, y, z0}, cp[3], cm[3];
        cp[0] = x + 1 == N ? 0 : x + 1;
        cm[0] = x == 0 ? N - 1 : x - 1;
        cp[1] = y + 1 == N ? 0 : y + 1;
        cm[1] = y == 0 ? N - 1 : y - 1;
        for (int s = 0; s < z1 - z0; ++s) {
            const int z = g.down ? z1 - 1 - s : z0 + s;
            c[2] = z;
            cp[2] = z + 1 == N ? 0 : z + 1;
            cm[2] = z == 0 ? N - 1 : z - 1;
            su2_site<MODE, NQ, STREAM>(g, wt, c, cp, cm, acc);
        }
    }

    if constexpr (MODE == kSU2Energy || MODE == kSU2KickSums) {
        u1_block_sums(acc, lds_red, &g.partials[(size_t)lid * NQ]);
    }
}

}  // namespace lat

namespace lat {

// Plain arrays to per-site records of the doublet and the links (kSU2StepAoS; the last
// pass of a call writes the plain arrays itself, kSU2StepOut):
// a[0..3] the doublet components, a[4 + 4 i + k] component k of link i;
// r[0] the doublet records, r[1 + i] those of link i.
struct SU2Soa {
    double *a[16];
};
struct SU2Aos {
    double4 *r[4];
};

__global__ void su2_to_aos(const SU2Soa s, const SU2Aos d, size_t V)
{
    for (size_t n = (size_t)blockIdx.x * blockDim.x + threadIdx.x; n < V; n += (size_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            d.r[q][n] = double4{s.a[4 * q][n], s.a[4 * q + 1][n], s.a[4 * q + 2][n], s.a[4 * q + 3][n]};
    }
}

}  // namespace lat
