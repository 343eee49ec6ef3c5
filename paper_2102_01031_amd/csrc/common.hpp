// common.hpp -- device-side records shared by the kernels and the runtime.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lat {

// Coefficients of one stencil pass at a kick point p of the schedule.
//   drift on load   phi += dload * pi            (the drift that ends at p)
//   kernel          F = ka1 * Lap(phi) - ka3 * dV/dphi       ka1 = a^{1+alpha}, ka3 = a^{3+alpha}
//   kicks           pi += c1 * F  (momenta now at p: energies sampled here)  pi += c2 * F
//   drift at end    phi += dend * pi            (leapfrog, local drift)
// Self-consistent expansion: the last block of pass p fills ka1, ka3, dload of
// pass p+1 from the energies it reduced (see ScaleRecord).
struct PassCoef {
    double ka1, ka3;
    double dload;
    double c1, c2;
    double dend;
    double h;       // sub-step leaving this kick point (0 at the last point)
    double cL, cR;  // weights of the two half kicks of b at this point
    double t;       // time at this kick point
    double t_next;  // time at the next kick point
    double *traj;   // if set, the update at this point stores (a, b) here: a at the
                    // point and b after its left half kick (integer time for VV2)
};

// Scale factor record on the device (self-consistent expansion) and the raw
// volume sums of the last reducing pass.
constexpr int kMaxQ = 16;
struct ScaleRecord {
    double a, b, t;
    double pad;
    double sums[kMaxQ];
    double maxes[4];
    double w[8];    // U(1) pass weights written on the device (self-consistent expansion)
};

// kLastSelf: velocity-Verlet update of b and a (self_update); kLastSelfLF:
// leapfrog update (self_update_lf), which also keeps the raw sums of the
// kicked momenta squared in ScaleRecord::sums[kPiPrev + f] for the next kick.
enum LastMode : int { kLastStore = 0, kLastSelf = 1, kLastSelfLF = 2 };
constexpr int kPiPrev = 8;

// Exchanges between the lanes of a wave on the vector unit, for reductions: each
// step pairs a lane with the one its group of 2, 4, 8, 16, 32 or 64 lanes still
// lacks, and both add the same two values, so all lanes end with the same bits.
// A step costs a few cycles of move and add latency, where a shuffle through the
// LDS crossbar waits for its return; the kernels that end or begin with sums are
// bound by that latency on small lattices (two float64 fields' self-consistent
// velocity-Verlet step: 32^3 10.4 -> 8.4 us, 96^3 23.5 -> 21.4 us).
template <int CTRL>
__device__ __forceinline__ double lane_dpp(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// v of this lane and of the lane 16 (SPAN = 16) or 32 lanes across: in *a that of
// the lower half of the pair of rows, in *b that of the upper
template <int SPAN>
__device__ __forceinline__ void lane_swap(double v, double *a, double *b)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    if constexpr (SPAN == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        *a = __hiloint2double((int)h[0], (int)l[0]);
        *b = __hiloint2double((int)h[1], (int)l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        *a = __hiloint2double((int)h[0], (int)l[0]);
        *b = __hiloint2double((int)h[1], (int)l[1]);
    }
}

// op over the wave's 64 lanes, the result in every lane (all lanes active)
template <typename OP>
__device__ __forceinline__ double wave_reduce(double v, OP &&op)
{
    double a, b;
    v = op(v, lane_dpp<0xB1>(v));    // quad_perm [1, 0, 3, 2]
    v = op(v, lane_dpp<0x4E>(v));    // quad_perm [2, 3, 0, 1]
    v = op(v, lane_dpp<0x141>(v));   // row_half_mirror
    v = op(v, lane_dpp<0x140>(v));   // row_mirror
    lane_swap<16>(v, &a, &b);
    v = op(a, b);
    lane_swap<32>(v, &a, &b);
    return op(a, b);
}

__device__ inline double wave_sum(double v)
{
    return wave_reduce(v, [](double x, double y) { return x + y; });
}

__device__ inline double wave_max(double v)
{
    return wave_reduce(v, [](double x, double y) { return fmax(x, y); });
}

__device__ inline void store_agent(double *p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline double load_agent(const double *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A block's arrival at a last-block reduction, called by the thread that stored
// the block's partials: the ticket increment releases them at agent scope, and
// only the block that takes the last ticket then acquires.  An agent-scope
// acquire invalidates the XCD's L2, so taking it in every block would throw out
// the neighbour planes that the other blocks on that XCD still read.  The
// acquire fence after the increment that read the final count synchronises with
// every block's release (the increments form one release sequence).
__device__ inline bool ticket_arrive(unsigned *ticket, unsigned nblocks)
{
    const unsigned prev = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    if (prev != nblocks - 1) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return true;
}

// Logical block id from the hardware block id: consecutive hardware blocks are
// dealt round-robin to the 8 XCDs, so give each XCD a contiguous range of
// logical tiles (neighbouring tiles then share that XCD's L2).
// Element access through a 32-bit byte offset from a uniform base pointer
// (valid while N^3 * sizeof(T) < 2^32, i.e. N <= 256 in float64).  Forming the
// offset in 32 bits lets the compiler use the scalar-base + 32-bit-offset
// global load and store forms, so every array shares one offset register
// instead of holding a 64-bit address per access.
template <typename T>
__device__ __forceinline__ T ld32(const T *base, unsigned i)
{
    return *(const T *)((const char *)base + (size_t)(i * (unsigned)sizeof(T)));
}

template <typename T>
__device__ __forceinline__ void st32(T *base, unsigned i, T v)
{
    *(T *)((char *)base + (size_t)(i * (unsigned)sizeof(T))) = v;
}

template <typename T>
__device__ __forceinline__ void st32_nt(T *base, unsigned i, T v)
{
    __builtin_nontemporal_store(v, (T *)((char *)base + (size_t)(i * (unsigned)sizeof(T))));
}

__device__ inline int xcd_logical_block(int b, int nb)
{
    const int per = nb / 8, rem = nb % 8;
    const int x = b % 8, j = b / 8;
    return x * per + (x < rem ? x : rem) + j;
}

// Block-wide deterministic sum of NQ values per thread into out[] (valid in the
// first wave).  No branch between the wave sums: their chains overlap.
template <int NT, int NQ>
__device__ inline void block_sums(double (&acc)[NQ], double *lds_red, double (&out)[NQ])
{
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    double v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = wave_sum(acc[q]);
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) lds_red[w * NQ + q] = v[q];
    }
    __syncthreads();
    if (tid < 64) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < NW; ++i) s += lds_red[i * NQ + q];
            out[q] = s;
        }
    }
    __syncthreads();
}

}  // namespace lat
