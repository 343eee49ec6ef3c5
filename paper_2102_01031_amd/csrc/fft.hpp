// fft.hpp -- power spectra of real N^3 fields without a library transform: three
// passes of line transforms in LDS, the last of which bins its result instead of
// storing it.
//
// Unnormalised forward DFT, sign e^{-i}, as a half spectrum F[(z N + y) HP + kx],
// kx in [0, N/2], rows padded to HP (a multiple of 8) so that eight neighbouring
// columns are one aligned 128-byte piece.
//   x pass   two real rows of one field per complex line of length N, separated by
//            the symmetry of real transforms: A(k) = (Z(k) + Z*(N-k))/2, B(k) = (Z(k) - Z*(N-k))/(2i)
//   y pass   eight columns of a plane per block, in place
//   z pass   eight columns per block; |F|^2 and mode counts go to the block's bins
// A pass reads and writes the spectrum once, and the last one only reads it: at 256^3 in
// float64 one spectrum moves 0.70 GB.  The y pass runs at memory's rate (6.0 TB/s); the x
// passes (3.9, with the combination 3.7) share their time with LDS, four conflict cycles to
// each of its instructions; the z pass (1.9) is bound by binning, one shell index and
// one LDS atomic per mode.
// Lines are transformed by Stockham's self-sorting algorithm with radices 8, 4, 2,
// 3, 5 and 7 (a plain sum per output for larger primes, between two buffers after a
// copy into LDS), one butterfly per thread and stage where a block has the threads, so
// that a stage can write over the LDS buffer it read (half the LDS of two buffers,
// twice the blocks per CU); the first stage reads its points from memory and the
// last stage of the y pass writes them without another trip through LDS.  At 256^3
// in float64: x pass 72 us (99 with two buffers and every stage through LDS; of the
// combination of two arrays 112), y pass 48 (92), z pass 77 (101), 0.70 GB in all; the
// library transform, its input copy and a binning pass took 270 us.  The roots of unity come from a
// table computed on the host in extended precision.
#pragma once
#include "common.hpp"
#include "fft_launch.hpp"

namespace lat {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return double2{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return double2{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return double2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
__device__ __forceinline__ double2 cmi(double2 a) { return double2{a.y, -a.x}; }   // -i a

// v[q] <- sum_p v[p] exp(-2 pi i p q / R)
template <int R>
__device__ __forceinline__ void dft(double2 (&v)[R])
{
    if constexpr (R == 1) {
        (void)v;
    } else if constexpr (R == 2) {
        const double2 a = v[0];
        v[0] = cadd(a, v[1]);
        v[1] = csub(a, v[1]);
    } else if constexpr (R == 4) {
        const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = cmi(csub(v[1], v[3]));
        v[0] = cadd(a, c);
        v[1] = cadd(b, d);
        v[2] = csub(a, c);
        v[3] = csub(b, d);
    } else if constexpr (R == 8) {
        constexpr double h = 0.70710678118654752440;
        double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft<4>(e);
        dft<4>(o);
        o[1] = double2{h * (o[1].x + o[1].y), h * (o[1].y - o[1].x)};
        o[2] = cmi(o[2]);
        o[3] = double2{h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y)};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = cadd(e[q], o[q]);
            v[q + 4] = csub(e[q], o[q]);
        }
    } else {
        // odd R: v0 + sums and differences of the pairs (p, R - p)
        static_assert(R == 3 || R == 5 || R == 7, "radix");
        // cos and sin of 2 pi j / R
        constexpr double C3[3] = {1.0, -0.5, -0.5}, S3[3] = {0.0, 0.86602540378443864676, -0.86602540378443864676};
        constexpr double C5[5] = {1.0, 0.30901699437494742410, -0.80901699437494742410, -0.80901699437494742410,
                                  0.30901699437494742410};
        constexpr double S5[5] = {0.0, 0.95105651629515357212, 0.58778525229247312917, -0.58778525229247312917,
                                  -0.95105651629515357212};
        constexpr double C7[7] = {1.0, 0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624,
                                  -0.90096886790241912624, -0.22252093395631440429, 0.62348980185873353053};
        constexpr double S7[7] = {0.0, 0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048,
                                  -0.43388373911755812048, -0.97492791218182360702, -0.78183148246802980871};
        constexpr int M = (R - 1) / 2;
        double2 s[M], d[M];
        double2 t = v[0];
#pragma unroll
        for (int p = 0; p < M; ++p) {
            s[p] = cadd(v[p + 1], v[R - 1 - p]);
            d[p] = csub(v[p + 1], v[R - 1 - p]);
            t = cadd(t, s[p]);
        }
        const double2 v0 = v[0];
        v[0] = t;
#pragma unroll
        for (int q = 1; q <= M; ++q) {
            double2 a = v0, b{0.0, 0.0};
#pragma unroll
            for (int p = 0; p < M; ++p) {
                const int j = (q * (p + 1)) % R;
                const double c = R == 3 ? C3[j % 3] : R == 5 ? C5[j % 5] : C7[j % 7];
                const double w = R == 3 ? S3[j % 3] : R == 5 ? S5[j % 5] : S7[j % 7];
                a.x += c * s[p].x;
                a.y += c * s[p].y;
                b.x += w * d[p].x;
                b.y += w * d[p].y;
            }
            const double2 mb = cmi(b);
            v[q] = cadd(a, mb);
            v[R - q] = csub(a, mb);
        }
    }
}

// LDS place of point i of a line in the x pass: one element skipped after every 16,
// so that the first stage's writes, eight points apart between neighbouring threads,
// meet all banks (fft_x at 256^3: 78 against 69 us).  In the column tiles eight lines
// lie side by side among the threads, and the line pitch alone spreads them.
template <bool COLS>
__device__ __forceinline__ unsigned fft_slot(unsigned i)
{
    return COLS ? i : i + (i >> 4);
}

// Butterfly j of line l: x[j + q M], q < R, M = N / R, times the stage's roots,
// transformed to y[(j / Ns) Ns R + j % Ns + q Ns].  Roots 1, 2 and 4 of the stage
// come from the table, the others are their products.
template <int R, typename LD>
__device__ __forceinline__ void butterfly(const FftPlan &P, unsigned Ns, unsigned j, const double2 *tw, LD ld,
                                          double2 (&v)[R], unsigned &o)
{
    const unsigned M = (unsigned)P.N / R;
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = ld(j + q * M);
    o = j * R;
    if (Ns > 1) {
        const unsigned jq = j / Ns, k = j - jq * Ns, s = k * ((unsigned)P.N / (Ns * R));
        o = jq * Ns * R + k;
        double2 w[R];
#pragma unroll
        for (int q = 1; q < R; ++q) {
            w[q] = (q & (q - 1)) == 0 ? tw[q * s] : cmul(w[q < 4 ? 2 : 4 % R], w[q < 4 ? 1 : q - 4]);
            v[q] = cmul(v[q], w[q]);
        }
    }
    dft<R>(v);
}

// One Stockham stage.  The block's threads cover the lines' butterflies, either all
// at once (P.inplace: every read happens before the first write, so `in` and `out`
// may be the same LDS buffer) or in a loop (between two buffers).  COLS: eight
// lines, line fastest among the threads (column tiles); else butterfly fastest.
template <int R, bool COLS, typename LD, typename ST>
__device__ __forceinline__ void fft_stage(const FftPlan &P, unsigned Ns, unsigned lines, const double2 *tw, LD ld,
                                          ST st)
{
    const unsigned M = (unsigned)P.N / R, total = lines * M;
    auto split = [&](unsigned b, unsigned &l, unsigned &j) {
        l = COLS ? b % kFftCols : b / M;
        j = COLS ? b / kFftCols : b - l * M;
    };
    double2 v[R];
    unsigned l = 0, j = 0, o = 0;
    if (P.inplace) {
        const bool on = threadIdx.x < total;
        if (on) {
            split(threadIdx.x, l, j);
            butterfly<R>(P, Ns, j, tw, [&](unsigned i) { return ld(l, i); }, v, o);
        }
        __syncthreads();
        if (on) {
#pragma unroll
            for (int q = 0; q < R; ++q) st(l, o + q * Ns, v[q]);
        }
    } else {
        for (unsigned b = threadIdx.x; b < total; b += blockDim.x) {
            split(b, l, j);
            butterfly<R>(P, Ns, j, tw, [&](unsigned i) { return ld(l, i); }, v, o);
#pragma unroll
            for (int q = 0; q < R; ++q) st(l, o + q * Ns, v[q]);
        }
    }
    __syncthreads();
}

// A stage of odd radix r, its sums taken over the r points as they lie in LDS (never
// in place): for the prime factors above 7, which have no butterfly of their own.  In
// a first stage (no roots on its points) a thread takes outputs q and r - q of a
// butterfly, which share the sums and differences of the points p and r - p; one
// output per thread and turn otherwise.  r / 2 complex products per output: a 61^3
// transform's three passes cost less than their launches, a spectrum and an occupation
// number of a 251^3 field 4.2 ms (7.0 with single outputs, 4.5 with the library).
template <bool COLS, typename LD, typename ST>
__device__ __forceinline__ void fft_stage_prime(unsigned r, const FftPlan &P, unsigned Ns, unsigned lines,
                                                const double2 *tw, LD ld, ST st)
{
    const unsigned N = (unsigned)P.N, M = N / r;
    if (Ns == 1) {
        const unsigned h = (r + 1) / 2, per = M * h, total = lines * per;
        for (unsigned b = threadIdx.x; b < total; b += blockDim.x) {
            const unsigned l = COLS ? b % kFftCols : b / per, e = COLS ? b / kFftCols : b - l * per;
            const unsigned j = e / h, q = e - j * h;
            double2 A = ld(l, j), B{0.0, 0.0};
            unsigned t = 0;
#pragma unroll 4
            for (unsigned p = 1; p < h; ++p) {
                t += q * M;
                if (t >= N) t -= N;
                const double2 x = ld(l, j + p * M), y = ld(l, j + (r - p) * M), w = tw[t];
                A.x += w.x * (x.x + y.x);
                A.y += w.x * (x.y + y.y);
                B.x += w.y * (x.x - y.x);
                B.y += w.y * (x.y - y.y);
            }
            st(l, j * r + q, double2{A.x - B.y, A.y + B.x});
            if (q) st(l, j * r + r - q, double2{A.x + B.y, A.y - B.x});
        }
    } else {
        const unsigned total = lines * N;
        for (unsigned b = threadIdx.x; b < total; b += blockDim.x) {
            const unsigned l = COLS ? b % kFftCols : b / N, o = COLS ? b / kFftCols : b - l * N;
            // output o = (j / Ns) Ns r + j % Ns + q Ns of butterfly j
            const unsigned hi = o / (Ns * r), rest = o - hi * (Ns * r), q = rest / Ns, k = rest - q * Ns;
            const unsigned j = hi * Ns + k, step = k * (N / (Ns * r)) + q * M;   // root of point p: tw[p step]
            double2 acc = ld(l, j);
            unsigned t = 0;
            for (unsigned p = 1; p < r; ++p) {
                t += step;
                if (t >= N) t -= N;
                acc = cadd(acc, cmul(ld(l, j + p * M), tw[t]));
            }
            st(l, o, acc);
        }
    }
    __syncthreads();
}

template <bool COLS, typename LD, typename ST>
__device__ __forceinline__ void fft_any(int r, const FftPlan &P, unsigned Ns, unsigned lines, const double2 *tw, LD ld,
                                        ST st)
{
    switch (r) {
    case 8: fft_stage<8, COLS>(P, Ns, lines, tw, ld, st); break;
    case 4: fft_stage<4, COLS>(P, Ns, lines, tw, ld, st); break;
    case 2: fft_stage<2, COLS>(P, Ns, lines, tw, ld, st); break;
    case 3: fft_stage<3, COLS>(P, Ns, lines, tw, ld, st); break;
    case 5: fft_stage<5, COLS>(P, Ns, lines, tw, ld, st); break;
    case 7: fft_stage<7, COLS>(P, Ns, lines, tw, ld, st); break;
    case 1: fft_stage<1, COLS>(P, Ns, lines, tw, ld, st); break;
    default: fft_stage_prime<COLS>((unsigned)r, P, Ns, lines, tw, ld, st); break;
    }
}

// Transform of `lines` lines: the first stage reads through `in`, the last one
// writes through `out`, the stages between them through LDS: first into b, then from
// b into a, and so on (a == b if P.inplace).  Every thread of the block calls it.
template <bool COLS, typename LD, typename ST>
__device__ __forceinline__ void fft_lines(const FftPlan &P, unsigned lines, const double2 *tw, double2 *a, double2 *b,
                                          LD in, ST out)
{
    const unsigned pitch = (unsigned)(COLS ? P.pitch : P.xpitch);
    auto rd = [&](unsigned l, unsigned i) { return a[l * pitch + fft_slot<COLS>(i)]; };
    auto wr = [&](unsigned l, unsigned i, double2 v) { b[l * pitch + fft_slot<COLS>(i)] = v; };
    if (P.nst == 1) {
        fft_any<COLS>(P.rad[0], P, 1, lines, tw, in, out);
        return;
    }
    fft_any<COLS>(P.rad[0], P, 1, lines, tw, in, wr);
    unsigned Ns = (unsigned)P.rad[0];
    for (int s = 1; s + 1 < P.nst; ++s) {
        double2 *t = a;
        a = b;
        b = t;
        fft_any<COLS>(P.rad[s], P, Ns, lines, tw, rd, wr);
        Ns *= (unsigned)P.rad[s];
    }
    a = b;
    fft_any<COLS>(P.rad[P.nst - 1], P, Ns, lines, tw, rd, out);
}

// x pass: rows 2 l and 2 l + 1 of f0 (MIX: of c0 f0 + c1 f1) make line l, P.lines lines
// per block.  A complex line's rounding follows its larger row, so both rows are one
// array's: with a row of phi and one of its momentum in a line, a momentum of 1e-8 phi
// kept nine digits.
template <typename T, bool MIX>
__global__ void __launch_bounds__(kFftMaxThreads) __attribute__((amdgpu_waves_per_eu(4)))
fft_x(const T *__restrict__ f0, const T *__restrict__ f1, double c0, double c1, double2 *__restrict__ G, const FftPlan P)
{
    extern __shared__ double2 fft_lds[];
    double2 *tw = fft_lds, *a = tw + P.N;
    double2 *b = a + (P.inplace ? 0 : P.lines * P.xpitch);
    double2 *z = P.nst % 2 == 0 ? a : b;                  // the last stage's result
    const unsigned N = (unsigned)P.N, rows = N * N, nl = (rows + 1) / 2;
    const unsigned l0 = blockIdx.x * (unsigned)P.lines;
    const unsigned mine = min((unsigned)P.lines, nl - l0);
    for (unsigned i = threadIdx.x; i < N; i += blockDim.x) tw[i] = P.tw[i];
    auto value = [&](size_t o) {
        double v = (double)f0[o];
        if constexpr (MIX) v = c0 * v + c1 * (double)f1[o];
        return v;
    };
    fft_lines<false>(
        P, mine, tw, a, b,
        [&](unsigned l, unsigned x) {
            const size_t r = 2 * (size_t)(l0 + l), o = r * N + x;
            return double2{value(o), r + 1 < rows ? value(o + N) : 0.0};
        },
        [&](unsigned l, unsigned i, double2 v) { z[l * P.xpitch + fft_slot<false>(i)] = v; });
    // whole padded rows (zeros past N / 2): no partly written pieces of memory
    const unsigned H = N / 2 + 1, HP = (unsigned)P.HP;
    for (unsigned e = threadIdx.x; e < mine * HP; e += blockDim.x) {
        const unsigned l = e / HP, k = e - l * HP;
        double2 A{0.0, 0.0}, B{0.0, 0.0};
        if (k < H) {
            const double2 p = z[l * P.xpitch + fft_slot<false>(k)], m = z[l * P.xpitch + fft_slot<false>(k == 0 ? 0 : N - k)];
            A = double2{0.5 * (p.x + m.x), 0.5 * (p.y - m.y)};
            B = double2{0.5 * (p.y + m.y), 0.5 * (m.x - p.x)};
        }
        const size_t r = 2 * (size_t)(l0 + l);
        G[r * HP + k] = A;
        if (r + 1 < rows) G[(r + 1) * HP + k] = B;
    }
}

// y pass in place: block (tile of kFftCols columns, plane z of G0 or, past N, of G1)
static __global__ void __launch_bounds__(kFftMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) fft_y(double2 *G0, double2 *G1, const FftPlan P)
{
    extern __shared__ double2 fft_lds[];
    double2 *tw = fft_lds, *a = tw + P.N;
    const int N = P.N, tiles = P.HP / kFftCols;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int tile = lid % tiles, zz = lid / tiles;
    double2 *G = (zz < N ? G0 : G1) + (size_t)(zz < N ? zz : zz - N) * N * P.HP + tile * kFftCols;
    for (int i = threadIdx.x; i < N; i += blockDim.x) tw[i] = P.tw[i];
    // the first stage's reads all happen before the last stage's writes (the LDS
    // stages between them, or the in-place stage's barrier)
    fft_lines<true>(
        P, kFftCols, tw, a, a + (P.inplace ? 0 : kFftCols * P.pitch),
        [&](unsigned l, unsigned i) { return G[i * (unsigned)P.HP + l]; },
        [&](unsigned l, unsigned i, double2 v) { G[i * (unsigned)P.HP + l] = v; });
}

// radial bin of a mode: the largest b with b^2 <= m (m < 2^24)
__device__ __forceinline__ int shell_of(int m)
{
    int b = (int)__builtin_amdgcn_sqrtf((float)m);   // within one of the root; settled below
    while ((b + 1) * (b + 1) <= m) ++b;
    while (b * b > m) --b;
    return b;
}

// z pass and binning.  Blocks loop over the N tiles ny x (HP / 8) column tiles of
// G0 (then of G1, if nq == 2), add w |F|^2 and the mode weights w (1, or 2 for a
// mode that stands for its mirror image too) to their bins in LDS, and leave one
// row per quantity: part[(q nbins + b) gridDim.x + block], q < nq sums, then the
// counts.  The transformed tile goes through LDS once more before the binning, which
// costs less than binning out of the last butterflies' registers (the index
// arithmetic of a whole butterfly at once spilled: 109 us at 256^3).
static __global__ void __launch_bounds__(kFftMaxThreads) __attribute__((amdgpu_waves_per_eu(4)))
fft_z_bin(const double2 *__restrict__ G0, const double2 *__restrict__ G1, int nq, const FftPlan P, int nbins,
          double *__restrict__ part)
{
    extern __shared__ double2 fft_lds[];
    double2 *tw = fft_lds, *a = tw + P.N;
    double2 *b = a + (P.inplace ? 0 : kFftCols * P.pitch), *res = P.nst % 2 == 0 ? a : b;   // res: the last stage's result
    double *bins = (double *)(a + (P.inplace ? 1 : 2) * kFftCols * P.pitch);            // [nq][nbins]
    unsigned *cnt = (unsigned *)(bins + nq * nbins);                                    // [nbins]
    const int N = P.N, tiles = P.HP / kFftCols, H = N / 2 + 1;
    const size_t plane = (size_t)N * P.HP;
    for (int i = threadIdx.x; i < N; i += blockDim.x) tw[i] = P.tw[i];
    for (int i = threadIdx.x; i < nq * nbins; i += blockDim.x) bins[i] = 0.0;
    for (int i = threadIdx.x; i < nbins; i += blockDim.x) cnt[i] = 0u;
    const int work = N * tiles * nq;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    for (int t = lid; t < work; t += gridDim.x) {
        const int q = t / (N * tiles), u = t - q * (N * tiles);
        const int tile = u % tiles, y = u / tiles;
        const double2 *G = (q ? G1 : G0) + (size_t)y * P.HP + tile * kFftCols;
        const int ny = y <= N / 2 ? y : y - N;
        __syncthreads();   // the bins' reset; the tile before has been read
        fft_lines<true>(
            P, kFftCols, tw, a, b, [&](unsigned l, unsigned i) { return G[i * plane + l]; },
            [&](unsigned l, unsigned i, double2 v) { res[l * P.pitch + i] = v; });
#pragma unroll 1
        for (int e = threadIdx.x; e < N * kFftCols; e += blockDim.x) {
            const int l = e % kFftCols, z = e / kFftCols, kx = tile * kFftCols + l;
            const int nz = z <= N / 2 ? z : z - N;
            const int bin = shell_of(kx * kx + ny * ny + nz * nz);
            if (kx >= H || bin >= nbins) continue;
            const unsigned w = (kx == 0 || 2 * kx == N) ? 1u : 2u;
            const double2 f = res[l * P.pitch + z];
            atomicAdd(&bins[q * nbins + bin], (double)w * (f.x * f.x + f.y * f.y));
            // the modes -ny and -nz lie in the same bin: a quarter of the modes counts them all
            if (q == 0 && 2 * y <= N && 2 * z <= N)
                atomicAdd(&cnt[bin], w * (y == 0 || 2 * y == N ? 1u : 2u) * (z == 0 || 2 * z == N ? 1u : 2u));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nq * nbins; i += blockDim.x) part[(size_t)i * gridDim.x + blockIdx.x] = bins[i];
    for (int i = threadIdx.x; i < nbins; i += blockDim.x)
        part[(size_t)(nq * nbins + i) * gridDim.x + blockIdx.x] = (double)cnt[i];
}

// Derivative of one bin's power with respect to the field, after the x and y passes:
// per tile the z transform, the modes of shell `bin` times `scale` and zeros for the
// others, conjugated, and the z transform again, in place in G; the y pass and
// fft_x_back then end at the real field, since a real field is the forward transform
// of its conjugated spectrum.  part[block]: the tile's share of the shell's power
// (w |F|^2, mirror modes counted).  Tiles that hold no mode of the shell are zeroed
// unread.
static __global__ void __launch_bounds__(kFftMaxThreads) __attribute__((amdgpu_waves_per_eu(4)))
fft_z_shell(double2 *__restrict__ G, const FftPlan P, int bin, double scale, double *__restrict__ part)
{
    extern __shared__ double2 fft_lds[];
    __shared__ double red[kFftMaxThreads / 64];
    double2 *tw = fft_lds, *a = tw + P.N;
    double2 *b = a + (P.inplace ? 0 : kFftCols * P.pitch), *res = P.nst % 2 == 0 ? a : b, *oth = res == a ? b : a;
    const int N = P.N, tiles = P.HP / kFftCols, H = N / 2 + 1;
    const size_t plane = (size_t)N * P.HP;
    const int lid = xcd_logical_block(blockIdx.x, gridDim.x);
    const int tile = lid % tiles, y = lid / tiles, ny = y <= N / 2 ? y : y - N;
    double2 *T = G + (size_t)y * P.HP + tile * kFftCols;
    // |k|^2 of the tile's modes lies between these two
    const int k0 = tile * kFftCols, k1 = min(k0 + kFftCols - 1, N / 2);
    const int lo = k0 * k0 + ny * ny, hi = k1 * k1 + ny * ny + (N / 2) * (N / 2);
    double acc = 0.0;
    if (lo < (bin + 1) * (bin + 1) && hi >= bin * bin) {
        for (int i = threadIdx.x; i < N; i += blockDim.x) tw[i] = P.tw[i];
        fft_lines<true>(
            P, kFftCols, tw, a, b, [&](unsigned l, unsigned i) { return T[i * plane + l]; },
            [&](unsigned l, unsigned i, double2 v) { res[l * P.pitch + i] = v; });
        for (int e = threadIdx.x; e < N * kFftCols; e += blockDim.x) {
            const int l = e % kFftCols, z = e / kFftCols, kx = k0 + l;
            const int nz = z <= N / 2 ? z : z - N;
            double2 f = res[l * P.pitch + z];
            if (kx < H && shell_of(kx * kx + ny * ny + nz * nz) == bin) {
                acc += (kx == 0 || 2 * kx == N ? 1.0 : 2.0) * (f.x * f.x + f.y * f.y);
                f = double2{scale * f.x, -scale * f.y};
            } else {
                f = double2{0.0, 0.0};
            }
            res[l * P.pitch + z] = f;
        }
        __syncthreads();
        fft_lines<true>(
            P, kFftCols, tw, res, oth, [&](unsigned l, unsigned i) { return res[l * P.pitch + i]; },
            [&](unsigned l, unsigned i, double2 v) { T[i * plane + l] = v; });
    } else {
        for (int e = threadIdx.x; e < N * kFftCols; e += blockDim.x)
            T[(size_t)(e / kFftCols) * plane + e % kFftCols] = double2{0.0, 0.0};
    }
    const double s = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < (int)(blockDim.x / 64); ++i) t += red[i];
        part[lid] = t;
    }
}

// Two real rows per complex line from their conjugated half spectra (fft_z_shell and
// the y pass after it): the line A + i B, whose upper half follows from the symmetry of
// real transforms, transforms to the rows a + i b.
static __global__ void __launch_bounds__(kFftMaxThreads) __attribute__((amdgpu_waves_per_eu(4)))
fft_x_back(const double2 *__restrict__ G, double *__restrict__ f, const FftPlan P)
{
    extern __shared__ double2 fft_lds[];
    double2 *tw = fft_lds, *a = tw + P.N;
    const unsigned N = (unsigned)P.N, rows = N * N, nl = (rows + 1) / 2;
    const unsigned l0 = blockIdx.x * (unsigned)P.lines;
    const unsigned mine = min((unsigned)P.lines, nl - l0);
    for (unsigned i = threadIdx.x; i < N; i += blockDim.x) tw[i] = P.tw[i];
    fft_lines<false>(
        P, mine, tw, a, a + (P.inplace ? 0 : P.lines * P.xpitch),
        [&](unsigned l, unsigned x) {
            const size_t r = 2 * (size_t)(l0 + l);
            const bool up = x > N / 2;
            const unsigned k = up ? N - x : x;
            const double sg = up ? -1.0 : 1.0;
            const double2 A = G[r * P.HP + k], B = r + 1 < rows ? G[(r + 1) * P.HP + k] : double2{0.0, 0.0};
            return double2{A.x - sg * B.y, sg * A.y + B.x};
        },
        [&](unsigned l, unsigned i, double2 v) {
            const size_t r = 2 * (size_t)(l0 + l);
            f[r * N + i] = v.x;
            if (r + 1 < rows) f[(r + 1) * N + i] = v.y;
        });
}

// out[row] = sum of the row's nb block values, one block per row, fixed order
static __global__ void __launch_bounds__(kFftThreads) spectrum_rows(const double *__restrict__ part, int nb,
                                                                    double *__restrict__ out)
{
    __shared__ double lds[kFftThreads / 64];
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += kFftThreads) s += part[(size_t)blockIdx.x * nb + i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < kFftThreads / 64; ++i) t += lds[i];
        out[blockIdx.x] = t;
    }
}

}  // namespace lat
