// fft_launch.hpp -- the line-transform plan and the spectrum passes' launchers
// (fft.hpp, fft_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace lat {

constexpr int kFftThreads = 256;   // of the row sums
constexpr int kFftMaxThreads = 512;
constexpr int kFftCols = 8;        // columns per block of the y and z passes
constexpr int kFftMaxN = 512;      // two buffers of eight lines fit 160 KB of LDS
constexpr int kFftMaxStages = 10;


struct FftPlan {
    int N, HP;
    int pitch, xpitch;             // pitch of a line in LDS (elements): column tiles, x pass
    int threads, lines;            // block size, lines per block of the x pass
    int inplace;                   // every stage's butterflies fit the block's threads
    int nst;
    int rad[kFftMaxStages];
    const double2 *tw;             // exp(-2 pi i k / N), k < N
};

constexpr int kFftBinBlocks = 1024; // blocks of the z pass (each leaves a row of bins)

// The stages for length N; false if N is too long, or too long for its largest prime
// factor.
bool fft_radices(int N, FftPlan *p);
// tw[k] = exp(-2 pi i k / N), k < N (host)
void fft_roots(int N, double2 *tw);

// Shell sums of |F|^2 of one real field f0 (nq = 1), or of f0 and c0 f0 + c1 f1
// (nq = 2): out[q nbins + b], then the mode counts out[nq nbins + b].  G0 and G1
// hold N^2 HP complex values each (G1 only for nq = 2), part (nq + 1) nbins
// kFftBinBlocks doubles; out may be pinned host memory.
hipError_t fft_spectra(const FftPlan &p, bool f32, const void *f0, const void *f1, double c0, double c1, int nq,
                       double2 *G0, double2 *G1, int nbins, double *part, double *out, hipStream_t st);

// Derivative of the power of shell `bin`, sum over its modes (mirror modes included)
// of |F|^2, with respect to the real field f0, times scale / 2: out[n] = scale times
// the inverse transform (unnormalised) of the shell's modes; *power = the shell sum.
// G as above, part N HP / kFftCols doubles.
hipError_t fft_shell_seed(const FftPlan &p, const double *f0, int bin, double scale, double2 *G, double *part,
                          double *power, double *out, hipStream_t st);

// out[r] = sum of part[r nb .. r nb + nb), r < rows, in a fixed order
hipError_t sum_rows(const double *part, int nb, int rows, double *out, hipStream_t st);

}  // namespace lat
