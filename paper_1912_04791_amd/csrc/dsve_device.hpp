// dsve_device.hpp -- device functions and the compile-time dispatch shared by the kernels of
// dsve_kernels.hip and dsve_resident.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dsve_dot.hpp"
#include "dsve_internal.hpp"
#include "dsve_math.hpp"

namespace dsve {

// Maximum over the 64 lanes of a wave of 32-bit values, read back to every lane.  DPP lane
// moves (swaps within quads, half-row and row mirrors: each lane then holds its row of 16; then
// the broadcasts of lane 15 of each row into the next row and of lane 31 into the upper half)
// leave the maximum in lane 63.  A lane whose DPP source lies outside the wave reads 0, the
// identity of the maximum, so every lane is written and no copy of the old value is needed.
template <int CTRL>
__device__ __forceinline__ unsigned dpp_umax32(unsigned v)
{
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
    return o > v ? o : v;
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v)
{
    v = dpp_umax32<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v = dpp_umax32<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v = dpp_umax32<0x141>(v);   // row_half_mirror
    v = dpp_umax32<0x140>(v);   // row_mirror
    v = dpp_umax32<0x142>(v);   // row_bcast:15
    v = dpp_umax32<0x143>(v);   // row_bcast:31
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
// Maximum over the wave of 64-bit patterns: the largest high word, then the largest low word among
// the lanes that hold it (one 32-bit maximum per step instead of a 64-bit compare and two selects).
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v)
{
    const unsigned hi = (unsigned)(v >> 32), lo = (unsigned)v;
    const unsigned mh = wave_max_u32(hi);
    const unsigned ml = wave_max_u32(hi == mh ? lo : 0u);
    return ((unsigned long long)mh << 32) | ml;
}

// Value of the lane below (lane 0 reads 0): one DPP move per 32-bit half.
__device__ __forceinline__ double lane_below(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x138, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Per-channel maximum of `v` (bit patterns of non-negative doubles, so unsigned order is
// value order and a NaN wins) over the active lanes of a wave.  Lanes are grouped by channel;
// a group whose channel is `home` goes to the workgroup accumulator in LDS, any other group
// straight to the global slot of its channel.
__device__ __forceinline__ void reduce_channel_max(unsigned long long v, int chan, bool active,
                                                   int home, unsigned long long *s_acc,
                                                   unsigned long long *gmax)
{
    const int lane = threadIdx.x & 63;
    unsigned long long pending = __ballot(active);
    while (pending) {
        const int leader = __ffsll((long long)pending) - 1;
        const int cl = __shfl(chan, leader, 64);
        const bool mine = active && (chan == cl);
        const unsigned long long m = wave_max_u64(mine ? v : 0ull);
        if (lane == leader) {
            if (cl == home) atomicMax(s_acc, m);
            else atomicMax(&gmax[cl], m);
        }
        pending &= ~__ballot(mine);
    }
}

// Atomic maximum of a workgroup's partial result into a per-channel slot, with `check` skipped when the
// slot already holds at least the value.  Slot values only grow while a kernel runs, so a load that
// returns an older (smaller) value only costs an atomic that was not needed; the load bypasses the
// compute unit's cache.  Most workgroups do not hold their channel's maximum, so most skip the atomic,
// which would otherwise serialise on the one address where many workgroups end together; but the
// workgroup waits for the load, and for the atomic alone it does not.
__device__ __forceinline__ void flush_max(unsigned long long *slot, unsigned long long v, bool check = true)
{
    if (check && v <= __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    (void)__hip_atomic_fetch_max(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// CFL maximum of channel c: the largest of its S sub-slots, as a double.  The floating-point
// maximum drops a NaN sub-slot when another holds a number; a NaN state still shows, since its
// cells stay NaN and the host's check of the last slot orders bit patterns as unsigned
// integers, where NaN is the largest.
__device__ __forceinline__ double amax_of(const unsigned long long *__restrict__ AM, int c,
                                         int64_t stride, int split)
{
    // every load goes out before the first is waited for (split is a power of two): one channel of 2^20
    // cells 20.6 -> 18.9 us a step, 100 000 cells 7.0 -> 6.4, against a branch and a wait per sub-slot
    double m = __longlong_as_double((long long)AM[c]);
    if (split > 1) {
        double v[kAmaxSplitMax];
#pragma unroll
        for (int s = 1; s < kAmaxSplitMax; ++s)
            v[s] = __longlong_as_double((long long)AM[c + (s & (split - 1)) * stride]);
#pragma unroll
        for (int s = 1; s < kAmaxSplitMax; ++s) m = fmax(m, v[s]);
    }
    return m;
}

__device__ __forceinline__ void raise_flag(unsigned int *flags, unsigned bad)
{
    if (bad) atomicOr(&flags[0], bad);
}

// Edge fluctuation and cell speed for the chosen precision and closure form.
template <int G, int PREC, int CL>
__device__ __forceinline__ void edge_fluct(double hL, double qL, double zL, double hR, double qR,
                                           double zR, double g, const Closure &K, double Dm[3],
                                           double Dp[3], unsigned &bad)
{
    if constexpr (PREC == PREC_FP64) fluct64<G, CL>(hL, qL, zL, hR, qR, zR, g, K, Dm, Dp, bad);
    else if constexpr (PREC == PREC_MIXED) fluct_mixed<G, CL>(hL, qL, zL, hR, qR, zR, g, K, Dm, Dp, bad);
    else fluct_dot<G, CL>(hL, qL, zL, hR, qR, zR, g, K, Dm, Dp, bad);
}

template <int PREC, int CL>
__device__ __forceinline__ double cell_speed(double h, double q, double g, const Closure &K,
                                             unsigned &bad)
{
    if constexpr (PREC == PREC_FP64) return speed64<CL>(h, q, g, K, bad);
    else if constexpr (PREC == PREC_MIXED) return speed_mixed<CL>(h, q, g, K, bad);
    else return speed_dot<CL>(h, q, g, K, bad);
}

// Ghost states (boundary conditions): the state beyond edge 0 (left) or edge N (right) of a
// channel from the adjacent cell's and the end's boundary data b = {h, q, z, dz/dt}.
__device__ __forceinline__ double ghost_h(int bc, const double *b, double h)
{
    return (bc == BC_FIXED_DEPTH || bc == BC_INFLOW_QH || bc == BC_DIRICHLET) ? b[0] : h;
}
__device__ __forceinline__ double ghost_q(int bc, const double *b, double q)
{
    return (bc == BC_INFLOW_Q || bc == BC_INFLOW_QH || bc == BC_DIRICHLET) ? b[1] : q;
}
__device__ __forceinline__ double ghost_z(int bc, const double *b, double z, double t)
{
    return bc == BC_DIRICHLET ? fma(t, b[3], b[2]) : z;
}

// Dispatch over the compile-time variants: G in [1, 5] quadrature points, closure (law).
#define DSVE_DISPATCH_G_CL(G, CL, MACRO)                                                  \
    switch ((G) * 8 + (CL)) {                                                             \
    case 8: MACRO(1, CL_GRASS); break;                                                \
    case 9: MACRO(1, CL_GRASS_THR); break;                                            \
    case 10: MACRO(1, CL_POWER); break;                                               \
    case 11: MACRO(1, CL_MPM); break;                                                 \
    case 12: MACRO(1, CL_VANRIJN); break;                                             \
    case 13: MACRO(1, CL_POWER_INT); break;                                           \
    case 16: MACRO(2, CL_GRASS); break;                                               \
    case 17: MACRO(2, CL_GRASS_THR); break;                                           \
    case 18: MACRO(2, CL_POWER); break;                                               \
    case 19: MACRO(2, CL_MPM); break;                                                 \
    case 20: MACRO(2, CL_VANRIJN); break;                                             \
    case 21: MACRO(2, CL_POWER_INT); break;                                           \
    case 24: MACRO(3, CL_GRASS); break;                                               \
    case 25: MACRO(3, CL_GRASS_THR); break;                                           \
    case 26: MACRO(3, CL_POWER); break;                                               \
    case 27: MACRO(3, CL_MPM); break;                                                 \
    case 28: MACRO(3, CL_VANRIJN); break;                                             \
    case 29: MACRO(3, CL_POWER_INT); break;                                           \
    case 32: MACRO(4, CL_GRASS); break;                                               \
    case 33: MACRO(4, CL_GRASS_THR); break;                                           \
    case 34: MACRO(4, CL_POWER); break;                                               \
    case 35: MACRO(4, CL_MPM); break;                                                 \
    case 36: MACRO(4, CL_VANRIJN); break;                                             \
    case 37: MACRO(4, CL_POWER_INT); break;                                           \
    case 40: MACRO(5, CL_GRASS); break;                                               \
    case 41: MACRO(5, CL_GRASS_THR); break;                                           \
    case 42: MACRO(5, CL_POWER); break;                                               \
    case 43: MACRO(5, CL_MPM); break;                                                 \
    case 44: MACRO(5, CL_VANRIJN); break;                                             \
    case 45: MACRO(5, CL_POWER_INT); break;                                           \
    default: return hipErrorInvalidValue;                                                 \
    }

// Dispatch over the closure alone.
#define DSVE_DISPATCH_CL(CL, MACRO)                                                       \
    switch (CL) {                                                                         \
    case CL_GRASS: MACRO(CL_GRASS); break;                                                \
    case CL_GRASS_THR: MACRO(CL_GRASS_THR); break;                                        \
    case CL_POWER: MACRO(CL_POWER); break;                                                \
    case CL_MPM: MACRO(CL_MPM); break;                                                    \
    case CL_VANRIJN: MACRO(CL_VANRIJN); break;                                            \
    case CL_POWER_INT: MACRO(CL_POWER_INT); break;                                        \
    default: return hipErrorInvalidValue;                                                 \
    }

}  // namespace dsve
