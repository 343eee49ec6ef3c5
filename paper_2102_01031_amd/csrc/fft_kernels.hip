// fft_kernels.hip -- launches of the spectrum passes (fft.hpp).
#include <algorithm>
#include <cmath>

#include "fft.hpp"

namespace lat {

bool fft_radices(int N, FftPlan *p)
{
    *p = FftPlan{};
    p->N = N;
    p->HP = (N / 2 + 1 + kFftCols - 1) / kFftCols * kFftCols;
    // a pitch of 2 mod 16 elements spreads the eight columns of a tile over the
    // LDS banks; in the x pass a line takes N + N / 16 elements (fft_slot)
    auto pitch = [](int len) { return len + ((2 - len) % 16 + 16) % 16; };
    p->pitch = pitch(N);
    p->xpitch = pitch(N + N / 16);
    if (N < 2 || N > kFftMaxN) return false;
    // powers of two: eights, with two fours in place of an eight and a two
    int n = N, two = 0, most = 0;
    while (n % 2 == 0) {
        n /= 2;
        ++two;
    }
    auto add = [&](int r) {
        if (p->nst < kFftMaxStages) p->rad[p->nst++] = r;
        most = std::max(most, kFftCols * (N / r));
    };
    for (; two > 4 || two == 3; two -= 3) add(8);
    for (; two >= 2; two -= 2) add(4);
    if (two) add(2);
    for (int r : {7, 5, 3})
        for (; n % r == 0; n /= r) add(r);
    p->threads = std::min(kFftMaxThreads, std::max(64, (most + 63) / 64 * 64));
    p->inplace = most <= p->threads;
    p->lines = kFftCols;
    if (n > 1) {
        // prime factors above 7: summed between two LDS buffers, after a stage of
        // radix 1 that brings the lines there.  Their cost grows with N r: spectrum and
        // occupation number 61^3 94 us (library transform 688), 251^3 2.6 ms (4.5),
        // 334 = 2 167 7.0 ms (7.0), 382 = 2 191 10.3 ms (9.4), 509^3 47 ms (35); the
        // library's plan costs 140 ms and more once per size besides
        int big[kFftMaxStages], nb = 0;
        for (int r = 11; n > 1 && nb < kFftMaxStages; r += 2)
            for (; n % r == 0 && nb < kFftMaxStages; n /= r) big[nb++] = r;
        if (n > 1 || N * big[nb - 1] > 65536 || p->nst + nb + 1 > kFftMaxStages) return false;
        for (int i = p->nst - 1; i >= 0; --i) p->rad[i + nb + 1] = p->rad[i];
        p->rad[0] = 1;
        for (int i = 0; i < nb; ++i) p->rad[1 + i] = big[i];
        p->nst += nb + 1;
        p->inplace = 0;
        p->threads = std::min(kFftMaxThreads, (kFftCols * (N + 1) / 2 + 63) / 64 * 64);
    }
    return true;
}

void fft_roots(int N, double2 *tw)
{
    const long double w = -2.0L * 3.14159265358979323846264338327950288L / N;
    for (int k = 0; k < N; ++k) tw[k] = double2{(double)std::cos(w * k), (double)std::sin(w * k)};
}

// dynamic LDS a pass may ask for (160 KB per CU; the kernels have little of their own)
constexpr int kFftLds = 156 * 1024;

template <typename F>
static hipError_t allow_lds(F fn)
{
    return hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, kFftLds);
}

static size_t lines_lds(const FftPlan &p, int pitch)
{
    return ((size_t)p.N + (size_t)(p.inplace ? 1 : 2) * kFftCols * pitch) * sizeof(double2);
}

template <typename T, bool MIX>
static hipError_t x_pass_of(const FftPlan &p, const void *f0, const void *f1, double c0, double c1, double2 *G,
                            hipStream_t st)
{
    const long nl = ((long)p.N * p.N + 1) / 2;
    const auto fn = fft_x<T, MIX>;
    const hipError_t e = allow_lds(fn);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, dim3((unsigned)((nl + p.lines - 1) / p.lines)), dim3(p.threads), lines_lds(p, p.xpitch), st,
                       (const T *)f0, (const T *)f1, c0, c1, G, p);
    return hipGetLastError();
}

// f0 to G0, and for nq = 2 the combination to G1
template <typename T>
static hipError_t x_pass(const FftPlan &p, const void *f0, const void *f1, double c0, double c1, int nq, double2 *G0,
                         double2 *G1, hipStream_t st)
{
    const hipError_t e = x_pass_of<T, false>(p, f0, nullptr, 1.0, 0.0, G0, st);
    return e != hipSuccess || nq == 1 ? e : x_pass_of<T, true>(p, f0, f1, c0, c1, G1, st);
}

hipError_t fft_spectra(const FftPlan &p, bool f32, const void *f0, const void *f1, double c0, double c1, int nq,
                       double2 *G0, double2 *G1, int nbins, double *part, double *out, hipStream_t st)
{
    hipError_t e = f32 ? x_pass<float>(p, f0, f1, c0, c1, nq, G0, G1, st)
                       : x_pass<double>(p, f0, f1, c0, c1, nq, G0, G1, st);
    if (e != hipSuccess) return e;
    const int tiles = p.N * (p.HP / kFftCols) * nq;
    if ((e = allow_lds(fft_y)) != hipSuccess || (e = allow_lds(fft_z_bin)) != hipSuccess) return e;
    hipLaunchKernelGGL(fft_y, dim3(tiles), dim3(p.threads), lines_lds(p, p.pitch), st, G0, G1, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int nb = std::min(tiles, kFftBinBlocks);
    const size_t lds = lines_lds(p, p.pitch) + (size_t)nq * nbins * sizeof(double) + (size_t)nbins * sizeof(unsigned);
    hipLaunchKernelGGL(fft_z_bin, dim3(nb), dim3(p.threads), lds, st, G0, G1, nq, p, nbins, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return sum_rows(part, nb, (nq + 1) * nbins, out, st);
}

hipError_t fft_shell_seed(const FftPlan &p, const double *f0, int bin, double scale, double2 *G, double *part,
                          double *power, double *out, hipStream_t st)
{
    hipError_t e = x_pass<double>(p, f0, nullptr, 0.0, 0.0, 1, G, nullptr, st);
    if (e != hipSuccess) return e;
    const int tiles = p.N * (p.HP / kFftCols);
    if ((e = allow_lds(fft_y)) != hipSuccess || (e = allow_lds(fft_z_shell)) != hipSuccess ||
        (e = allow_lds(fft_x_back)) != hipSuccess)
        return e;
    const size_t lds = lines_lds(p, p.pitch);
    hipLaunchKernelGGL(fft_y, dim3(tiles), dim3(p.threads), lds, st, G, (double2 *)nullptr, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(fft_z_shell, dim3(tiles), dim3(p.threads), lds, st, G, p, bin, scale, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = sum_rows(part, tiles, 1, power, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(fft_y, dim3(tiles), dim3(p.threads), lds, st, G, (double2 *)nullptr, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const long nl = ((long)p.N * p.N + 1) / 2;
    hipLaunchKernelGGL(fft_x_back, dim3((unsigned)((nl + p.lines - 1) / p.lines)), dim3(p.threads),
                       lines_lds(p, p.xpitch), st, (const double2 *)G, out, p);
    return hipGetLastError();
}

hipError_t sum_rows(const double *part, int nb, int rows, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(spectrum_rows, dim3(rows), dim3(kFftThreads), 0, st, part, nb, out);
    return hipGetLastError();
}

}  // namespace lat
