// dsve_kernels.hip -- HIP kernels of the A-DOT hot path for gfx950 (wave64).
//
// k_step      one fused kernel per time step: ghost cells (boundary conditions), DOT fluctuation of
//             every edge, exchange of D^+ with the lane above by a DPP lane move, cell update into
//             the other ping-pong buffer, CFL speed of the new state reduced per channel (DPP lane
//             moves -> LDS -> one global atomic max per workgroup into its CFL sub-slot).
// k_step_packed  the same for many short channels: tiles over the flat edge space of all channels.
// k_start     CFL maximum of the state a run starts from (k_cfl: the same for many short channels).
// k_cfl_one   CFL maximum and time step of one channel (cfl_reduce entry point).
// k_fluct     pairwise fluctuations (dot_edge_fluct entry point).
// k_update    cell update from given fluctuations (cell_update entry point).
//
// Every kernel comes in one closure form per bed-load law: CL_GRASS (the Grass law in closed
// form, the workloads of Sec. 4) and the other laws through b = xi dq_s/dq per state (Sec. 2,
// Sec. 5), and in three arithmetic forms: FP64 and mixed closed form (Sec. 3.3), and FP64 with
// the numerical eigen-decomposition of the original DOT solver (Sec. 3.1), the baseline of the
// closed form.
//
// Every cell is updated by exactly one thread and every value computed depends only on its own edge
// or cell, so results do not depend on the kernel, the workgroup size or the number of workgroups.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "dsve_device.hpp"

namespace dsve {

// Index arithmetic of the packed step kernel: 32-bit when the context has fewer than 2^29 edges (then
// every byte offset into a state array fits in 32 bits and a load is an SGPR base plus a 32-bit
// VGPR offset), 64-bit otherwise.
template <bool WIDE> struct StepIdx { using type = int32_t; };
template <> struct StepIdx<true> { using type = int64_t; };

template <bool WIDE, typename I>
__device__ __forceinline__ double ldx(const double *__restrict__ p, I i)
{
    if constexpr (WIDE) return p[i];
    else return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(p) + ((uint32_t)i << 3));
}
__device__ __forceinline__ double ldx(const double *__restrict__ p, int i)
{
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(p) + ((uint32_t)i << 3));
}
__device__ __forceinline__ void stx(double *__restrict__ p, int i, double v)
{
    *reinterpret_cast<double *>(reinterpret_cast<char *>(p) + ((uint32_t)i << 3)) = v;
}
template <bool WIDE, typename I>
__device__ __forceinline__ void stx(double *__restrict__ p, I i, double v)
{
    if constexpr (WIDE) p[i] = v;
    else *reinterpret_cast<double *>(reinterpret_cast<char *>(p) + ((uint32_t)i << 3)) = v;
}

// ---------------------------------------------------------------------------
// Step kernel for many short channels: a workgroup of T threads takes T consecutive edges of the flat
// edge space and updates the T-1 cells whose two faces both lie in the tile; tile k starts at edge
// k (T-1), so consecutive tiles share one edge, which both compute, and a tile holds several whole
// channels.  D^- goes to the left neighbour through LDS.
template <int G, int PREC, int CL, bool WIDE>
__global__ __launch_bounds__(kMaxTile, step_min_waves(PREC, CL)) void k_step_packed(StepArgs A, const ChanInfo *__restrict__ CH,
                                                                                  const int64_t *__restrict__ EO,
                                                                                  const int32_t *__restrict__ TC,
                                                                                  const unsigned long long *__restrict__ AM)
{
    extern __shared__ double s_dm_all[];      // [2][3][T]: D^- of even and odd tiles
    __shared__ unsigned long long s_acc;
    using Idx = typename StepIdx<WIDE>::type;
    const int T = blockDim.x;
    const int t = threadIdx.x;
    const int lane = t & 63;

    // Each workgroup takes a contiguous run of tiles (the tiles split evenly over the grid: lo or
    // lo + 1 per workgroup, from the host; tile indices fit 32 bits, the host refuses 2^31
    // tiles), so consecutive tiles mostly share their home channel, the channel of the tile's
    // first edge.  The home channel's values (edge offsets, boundary codes, CFL maximum of W^n,
    // time step) are loaded when the run enters the channel, and every lane keeps the running
    // CFL maximum of its cells in it; the lanes are reduced across only when the run leaves the
    // channel, and at the end.  Cells of another channel (a tile that straddles a channel's
    // end) find their channel by a forward scan and go to its slot at once.
    const int wg = (int)blockIdx.x;
    const int k_first = wg * A.tiles_lo + (wg < A.tiles_rem ? wg : A.tiles_rem);
    const int k_end = k_first + A.tiles_lo + (wg < A.tiles_rem ? 1 : 0);
    if (t == 0) s_acc = 0ull;
    if (k_first >= k_end) return;   // the same for the whole workgroup
    // this workgroup's sub-slot of the CFL maxima it merges into (S is a power of two)
    unsigned long long *const amax_mine =
        A.amax_next + (int64_t)(blockIdx.x & (unsigned)(A.amax_split - 1)) * A.amax_stride;
    int home = -1;
    Idx eo0 = 0, eo1 = 0;
    int h_bcl = 0, h_bcr = 0;
    double am_home = 0.0, dt_home = 0.0, r_home = 0.0;
    unsigned long long lane_acc = 0ull;
    int nx_home = TC[k_first];
    for (int k = k_first; k < k_end; ++k) {
        const int tile_home = nx_home;
        if (k + 1 < k_end) nx_home = TC[k + 1];
        if (tile_home != home) {
            if (home >= 0) {
                // merge what the lanes hold for the channel the run leaves (two barriers, once
                // per channel, not per tile)
                const unsigned long long m = wave_max_u64(lane_acc);
                if (lane == 0 && m != 0ull) atomicMax(&s_acc, m);
                __syncthreads();
                if (t == 0) {
                    if (s_acc != 0ull) flush_max(&amax_mine[home], s_acc);
                    s_acc = 0ull;
                }
                __syncthreads();
                lane_acc = 0ull;
            }
            // (a channel's first cell and length follow from its edge offsets: eoff[c] = off[c] + c)
            home = tile_home;
            eo0 = (Idx)EO[home];
            eo1 = (Idx)EO[home + 1];
            h_bcl = CH[home].bcl;
            h_bcr = CH[home].bcr;
            am_home = amax_of(AM, home, A.amax_stride, A.amax_split);
            // dt = CFL dx / amax and dt/dx, as every lane of another channel computes them
            dt_home = CH[home].cfl_dx * rcp_h(am_home);
            r_home = dt_home * CH[home].inv_dx;
        }
        const Idx h_cell0 = eo0 - home, h_ncell = eo1 - eo0 - 1;
        double *const s_dm = s_dm_all + (int)(k & 1) * 3 * T;
        // lanes past the last edge (in the last tile only) compute the last edge again: their
        // results are never stored and no lane that updates a cell reads them
        const Idx ge_raw = (Idx)k * (Idx)(T - 1) + t;
        const bool have_edge = ge_raw < (Idx)A.n_edges;
        const Idx ge = have_edge ? ge_raw : (Idx)A.n_edges - 1;
        int c = home;
        Idx eoc = eo0, cell0 = h_cell0, ncell = h_ncell;
        int bcl = h_bcl, bcr = h_bcr;
        if (ge >= eo1) {
            c = home + 1;
            while (ge >= (Idx)EO[c + 1]) ++c;
            eoc = (Idx)EO[c];
            cell0 = eoc - c;
            ncell = (Idx)EO[c + 1] - eoc - 1;
            bcl = CH[c].bcl;
            bcr = CH[c].bcr;
        }
        // the home channel's record is the same for the whole workgroup (scalar loads); lanes
        // of another channel load their own
        const ChanInfo hci = CH[home];
        ChanInfo ci = hci;
        if (c != home) ci = CH[c];
        const Closure K = closure_of(ci);
        const Idx e = ge - eoc;
        unsigned bad = 0u;
        double Dm[3], Dp[3];
        const Idx N = ncell, base = cell0;
        const Idx il = (e == 0) ? (bcl == BC_PERIODIC ? base + N - 1 : base) : base + e - 1;
        const Idx ir = (e == N) ? (bcr == BC_PERIODIC ? base : base + N - 1) : base + e;
        double hL = ldx<WIDE>(A.h, il);
        double qL = ldx<WIDE>(A.q, il);
        double zL = ldx<WIDE>(A.z, il);
        const double hR = ldx<WIDE>(A.h, ir);
        const double qR = ldx<WIDE>(A.q, ir);
        const double zR = ldx<WIDE>(A.z, ir);
        {
            double hRe = hR, qRe = qR, zRe = zR;
            if (e == 0) {
                hL = ghost_h(ci.bcl, ci.bl, hL);
                qL = ghost_q(ci.bcl, ci.bl, qL);
                if (ci.bcl == BC_DIRICHLET) zL = ghost_z(ci.bcl, ci.bl, zL, A.t_cur[c]);
            } else if (e == N) {
                hRe = ghost_h(ci.bcr, ci.br, hR);
                qRe = ghost_q(ci.bcr, ci.br, qR);
                if (ci.bcr == BC_DIRICHLET) zRe = ghost_z(ci.bcr, ci.br, zR, A.t_cur[c]);
            }
            edge_fluct<G, PREC, CL>(hL, qL, zL, hRe, qRe, zRe, A.g, K, Dm, Dp, bad);
        }
        // D^- goes to the left neighbour through this tile's half of the LDS buffer; the next
        // tile writes the other half, so one barrier per tile orders every write after the
        // reads of the tile before
        s_dm[t] = Dm[0];
        s_dm[T + t] = Dm[1];
        s_dm[2 * T + t] = Dm[2];
        __syncthreads();
        const bool upd = have_edge && (t < T - 1) && (e < ncell);
        unsigned long long sp_bits = 0ull;
        if (upd) {
            double dt = dt_home, r = r_home;
            if (c != home) {
                dt = ci.cfl_dx * rcp_h(amax_of(AM, c, A.amax_stride, A.amax_split));
                r = dt * ci.inv_dx;
            }
            const Idx i = cell0 + e;
            // W_i^{n+1} = W_i^n - dt/dx (D^-_{i+1/2} + D^+_{i-1/2}) + dt S(W_i^n)
            // (Sec. 3, Eq. scheme; S from the friction slope when K_s is given)
            const double hn = hR - r * (s_dm[t + 1] + Dp[0]);
            double qn = qR - r * (s_dm[T + t + 1] + Dp[1]);
            const double zn = zR - r * (s_dm[2 * T + t + 1] + Dp[2]);
            if (ci.fric > 0.0) qn = fma(dt, friction_source(hR, qR, A.g, ci.fric), qn);
            stx<WIDE>(A.hn, i, hn);
            stx<WIDE>(A.qn, i, qn);
            stx<WIDE>(A.zn, i, zn);
            const double sp = fabs(cell_speed<PREC, CL>(hn, qn, A.g, K, bad));
            sp_bits = (unsigned long long)__double_as_longlong(sp);
            if (e == 0) {
                A.t_next[c] = A.t_cur[c] + dt;
                A.amax_clear[c] = 0ull;
#pragma unroll
                for (int s = 1; s < kAmaxSplitMax; ++s)
                    if (s < A.amax_split) A.amax_clear[c + s * A.amax_stride] = 0ull;
            }
        }
        raise_flag(A.flags, bad);
        const bool mine = upd && c == home;
        lane_acc = (mine && sp_bits > lane_acc) ? sp_bits : lane_acc;
        const bool other = upd && c != home;
        if (__ballot(other)) reduce_channel_max(sp_bits, c, other, -1, &s_acc, amax_mine);
    }
    const unsigned long long m = wave_max_u64(lane_acc);
    if (lane == 0 && m != 0ull) atomicMax(&s_acc, m);
    __syncthreads();
    if (t == 0 && s_acc != 0ull) flush_max(&amax_mine[home], s_acc);
}

// ---------------------------------------------------------------------------
// Merges the lanes' maxima of a kernel of one segment per wave into the slots of their channels (-1: a
// wave without a segment): within the wave, then the waves of the workgroup in the same channel in LDS.
// Every thread of the workgroup calls it, once.
__device__ __forceinline__ void merge_max(unsigned long long acc, int c, unsigned long long *amax, int shift, bool check)
{
    __shared__ unsigned long long s_max[kMaxTile / 64];
    __shared__ int s_chan[kMaxTile / 64];
    const int t = (int)threadIdx.x, waves = (int)(blockDim.x >> 6);
    const unsigned long long m = wave_max_u64(acc);
    if (waves == 1) {
        if (t == 0 && c >= 0 && m != 0ull) flush_max(&amax[c << shift], m, check);
        return;
    }
    if ((t & 63) == 0) {
        s_max[t >> 6] = m;
        s_chan[t >> 6] = c;
    }
    __syncthreads();
    if (t < waves && s_chan[t] >= 0 && (t == 0 || s_chan[t - 1] != s_chan[t])) {
        unsigned long long v = s_max[t];
        for (int w = t + 1; w < waves && s_chan[w] == s_chan[t]; ++w) v = s_max[w] > v ? s_max[w] : v;
        if (v != 0ull) flush_max(&amax[s_chan[t] << shift], v, check);
    }
}

// Step kernel over segments: each wave takes one segment, a run of cells of one channel, in tiles of
// 64 edges (63 cells: the first edge of a tile is the last of the tile before, computed by both).
// Lane l computes edge e = t0 + l of the segment, the left face of cell e, and updates cell e - 1,
// whose right face it is, with D^+ of the edge below from the lane below.
//
// Waves share nothing until their CFL maxima are merged, so no wave waits for another at a tile, and
// everything of the channel is the same for the whole wave (scalar registers and branches; the lanes
// at a channel's ends fix up their ghost cell in a branch that other tiles skip).  Bound by VALU issue
// in FP64 and by the waits of each wave on its dependent instructions.  Against tiles of 256 edges with
// D^- through LDS, a barrier per tile and per-lane channel lookups, the same arithmetic (that of the
// time) took, FP64: 65 536 channels of 512-4096 cells 3.12 -> 2.47 ms a step, one channel of 2^20 cells
// 24.5 -> 22.3 us; mixed: one of 4 000 001 cells 65 -> 56 us.
template <int G, int PREC, int CL>
__global__ __launch_bounds__(kMaxTile, step_min_waves(PREC, CL)) void k_step(StepArgs A, const ChanInfo *__restrict__ CH,
                                                                           const Segment *__restrict__ SEG,
                                                                           const unsigned long long *__restrict__ AM)
{
    const int lane = threadIdx.x & 63;
    const int sidx = (int)blockIdx.x * (int)(blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned long long acc = 0ull;
    int c = -1;
    if (sidx < A.n_segments) {
        const Segment sg = SEG[sidx];
        const int n = (int)(sg.n_flags >> 2);
        const bool first = (sg.n_flags & 1u) != 0u, last = (sg.n_flags & 2u) != 0u;
        c = sg.chan;
        const ChanInfo &ci = CH[c];
        const Closure K = closure_of(ci);
        const double fric = ci.fric;
        // cell i of the segment is at index i + 1 from these bases (cell -1, the left neighbour of
        // a segment inside a channel, at 0; a segment at its channel's start does not read it)
        const int64_t base = sg.cell0 - 1;
        const double *const h = A.h + base, *const q = A.q + base, *const z = A.z + base;
        double *const hn = A.hn + base, *const qn = A.qn + base, *const zn = A.zn + base;
        const int il_min = first ? 1 : 0, ir_max = last ? n : n + 1;
        // FP64: each tile's states are under way while the tile before is computed, the first tile's
        // while the time step is formed (120 registers, still four waves a SIMD: 65 536 channels 1.92
        // -> 1.90 ms a step, 2^20 cells 19.9 -> 19.6 us).  Mixed keeps its fifth wave instead (99
        // registers with it, 93 without).
        struct Sides {
            double hL, qL, zL, hR, qR, zR;
        };
        const auto load = [&](int t) {
            // lanes past the segment's last edge compute it again; they update nothing
            const int e = t + lane < n ? t + lane : n;
            const int il = e > il_min ? e : il_min, ir = e + 1 < ir_max ? e + 1 : ir_max;
            return Sides{ldx(h, il), ldx(q, il), ldx(z, il), ldx(h, ir), ldx(q, ir), ldx(z, ir)};
        };
        Sides next;
        if constexpr (PREC == PREC_FP64) next = load(0);
        const double dt = ci.cfl_dx * rcp_h(amax_of(AM, c << A.amax_shift, A.amax_stride, A.amax_split));
        const double r = dt * ci.inv_dx;
        unsigned bad = 0u;
        for (int t0 = 0; t0 < n; t0 += kSegTile) {
            const int e = t0 + lane < n ? t0 + lane : n;
            if constexpr (PREC != PREC_FP64) next = load(t0);
            double hL = next.hL, qL = next.qL, zL = next.zL, hR = next.hR, qR = next.qR, zR = next.zR;
            if constexpr (PREC == PREC_FP64)
                if (t0 + kSegTile < n) next = load(t0 + kSegTile);
            const double h0 = hL, q0 = qL, z0 = zL;
            if (first && t0 == 0) {
                // ghost cell left of the channel's first cell (which every lane of edge 0 holds as R)
                double gh = hR, gq = qR, gz = zR;
                if (ci.bcl == BC_PERIODIC) {
                    const int64_t far = ci.cell0 + ci.ncell - 1;
                    gh = A.h[far];
                    gq = A.q[far];
                    gz = A.z[far];
                }
                gh = ghost_h(ci.bcl, ci.bl, gh);
                gq = ghost_q(ci.bcl, ci.bl, gq);
                if (ci.bcl == BC_DIRICHLET) gz = ghost_z(ci.bcl, ci.bl, gz, A.t_cur[c]);
                if (e == 0) {
                    hL = gh;
                    qL = gq;
                    zL = gz;
                }
            }
            if (last && t0 + 64 > n) {
                // ghost cell right of the channel's last cell
                double gh = h0, gq = q0, gz = z0;
                if (ci.bcr == BC_PERIODIC) {
                    gh = A.h[ci.cell0];
                    gq = A.q[ci.cell0];
                    gz = A.z[ci.cell0];
                }
                gh = ghost_h(ci.bcr, ci.br, gh);
                gq = ghost_q(ci.bcr, ci.br, gq);
                if (ci.bcr == BC_DIRICHLET) gz = ghost_z(ci.bcr, ci.br, gz, A.t_cur[c]);
                if (e == n) {
                    hR = gh;
                    qR = gq;
                    zR = gz;
                }
            }
            double Dm[3], Dp[3];
            edge_fluct<G, PREC, CL>(hL, qL, zL, hR, qR, zR, A.g, K, Dm, Dp, bad);
            const double p0 = lane_below(Dp[0]), p1 = lane_below(Dp[1]), p2 = lane_below(Dp[2]);
            if (lane > 0 && t0 + lane <= n) {
                // W_i^{n+1} = W_i^n - dt/dx (D^-_{i+1/2} + D^+_{i-1/2}) + dt S(W_i^n)
                // (Sec. 3, Eq. scheme; S from the friction slope when K_s is given)
                const double hv = h0 - r * (Dm[0] + p0);
                double qv = q0 - r * (Dm[1] + p1);
                const double zv = z0 - r * (Dm[2] + p2);
                if (fric > 0.0) qv = fma(dt, friction_source(h0, q0, A.g, fric), qv);
                stx(hn, e, hv);
                stx(qn, e, qv);
                stx(zn, e, zv);
                const double sp = fabs(cell_speed<PREC, CL>(hv, qv, A.g, K, bad));
                const unsigned long long bits = (unsigned long long)__double_as_longlong(sp);
                acc = bits > acc ? bits : acc;
            }
        }
        if (first && lane == 0) {
            A.t_next[c] = A.t_cur[c] + dt;
            const int at = c << A.amax_shift;
            A.amax_clear[at] = 0ull;
#pragma unroll
            for (int s = 1; s < kAmaxSplitMax; ++s)
                if (s < A.amax_split) A.amax_clear[at + s * A.amax_stride] = 0ull;
        }
        raise_flag(A.flags, bad);
    }
    unsigned long long *const amax_mine =
        A.amax_next + (int64_t)(blockIdx.x & (unsigned)(A.amax_split - 1)) * A.amax_stride;
    merge_max(acc, c, amax_mine, A.amax_shift, A.amax_check != 0);
}

// ---------------------------------------------------------------------------
__device__ __forceinline__ int find_channel(const int64_t *off, int C, int64_t i)
{
    int lo = 0, hi = C;   // off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Grid-stride over cells; each workgroup keeps its running maximum for one channel at a
// time and flushes it with one global atomic when the channel changes (cells are visited in
// increasing order within a workgroup, so channels change monotonically).
template <int PREC, int CL>
__global__ __launch_bounds__(kCflThreads) void k_cfl(CflArgs A)
{
    // Each workgroup takes a contiguous range of cells, kCflThreads at a time.  Every lane keeps
    // the running maximum of its cells in its wave's current channel `cur` (wave-uniform); the
    // lanes are reduced across only when one of them reaches another channel, and at the end.
    // The workgroup's home channel (that of its first cell) collects in LDS and is merged into
    // its slot once; other channels go to their slots directly.  Workgroups of 1024 threads keep
    // those end-of-kernel merges, which serialise on one address, to a few hundred.
    __shared__ unsigned long long s_acc;
    const int lane = threadIdx.x & 63;
    const int64_t per =
        ((A.n_cells + gridDim.x - 1) / gridDim.x + kCflThreads - 1) / kCflThreads * kCflThreads;
    const int64_t start = (int64_t)blockIdx.x * per;
    const int64_t end = start + per < A.n_cells ? start + per : A.n_cells;
    if (threadIdx.x == 0) s_acc = 0ull;
    __syncthreads();
    if (start >= end) return;   // the same for the whole workgroup
    const int home = find_channel(A.off, A.n_channels, start);
    int c = home;                  // channel of this lane's cell
    int cur = home;                // the wave's current channel
    unsigned long long acc = 0ull; // this lane's maximum over its cells in `cur`
    unsigned bad = 0u;
    // the lane's channel end and closure stay in registers until the lane leaves the channel,
    // so the common iteration waits only for its own cell's state
    int64_t c_end = A.off[c + 1];
    Closure K = closure_of(A.ch[c]);
    for (int64_t i0 = start; i0 < end; i0 += kCflThreads) {
        const int64_t i = i0 + threadIdx.x;
        const bool active = i < end;
        unsigned long long bits = 0ull;
        if (active) {
            if (i >= c_end) {
                do {
                    ++c;
                    c_end = A.off[c + 1];
                } while (i >= c_end);
                K = closure_of(A.ch[c]);
            }
            const double sp = fabs(cell_speed<PREC, CL>(A.h[i], A.q[i], A.g, K, bad));
            bits = (unsigned long long)__double_as_longlong(sp);
        }
        const unsigned long long moved = __ballot(active && c != cur);
        if (moved == 0ull) {
            if (active) acc = bits > acc ? bits : acc;
        } else {
            // the wave leaves `cur`: merge what its lanes hold for it, then this round's cells
            // by channel, and go on in the channel of its last active lane
            const unsigned long long m = wave_max_u64(acc);
            if (lane == 0 && m != 0ull) {
                if (cur == home) atomicMax(&s_acc, m);
                else flush_max(&A.amax[cur], m);
            }
            acc = 0ull;
            reduce_channel_max(bits, c, active, home, &s_acc, A.amax);
            const unsigned long long act = __ballot(active);
            cur = __shfl(c, 63 - __clzll((long long)act), 64);
        }
    }
    const unsigned long long m = wave_max_u64(acc);
    if (lane == 0 && m != 0ull) {
        if (cur == home) atomicMax(&s_acc, m);
        else flush_max(&A.amax[cur], m);
    }
    raise_flag(A.flags, bad);
    __syncthreads();
    if (threadIdx.x == 0 && s_acc != 0ull) flush_max(&A.amax[home], s_acc);
}

// Speeds of cells base + [0, n) of a channel, kAhead cells per lane at a time so that their loads are in
// flight together; each(i, h, q) sees every cell read.
constexpr int kAhead = 4;
template <int PREC, int CL, typename F>
__device__ __forceinline__ unsigned long long speeds_of(const double *h, const double *q, int n, double g,
                                                        const Closure &K, unsigned &bad, F each)
{
    const int lane = threadIdx.x & 63;
    unsigned long long acc = 0ull;
    for (int i0 = 0; i0 < n; i0 += 64 * kAhead) {
        double hv[kAhead], qv[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            // lanes past the end read the last cell again
            const int i = i0 + 64 * k + lane < n ? i0 + 64 * k + lane : n - 1;
            hv[k] = ldx(h, i);
            qv[k] = ldx(q, i);
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (i0 + 64 * k >= n) break;
            each(i0 + 64 * k + lane < n ? i0 + 64 * k + lane : n - 1, hv[k], qv[k]);
            const unsigned long long b =
                (unsigned long long)__double_as_longlong(fabs(cell_speed<PREC, CL>(hv[k], qv[k], g, K, bad)));
            acc = b > acc ? b : acc;
        }
    }
    return acc;
}

// Start of a run over segments: the CFL maximum of the state per channel and, for a run of an odd number
// of steps, which then ends in the caller's arrays, the copy of state and clocks that it starts from.
//
// Bound by HBM (16 B a cell, 48 with the copy).  Workgroups of 1024 threads over contiguous ranges, one
// cell per lane in flight, took 895 us for 151 M cells (2.7 TB/s), and the copies after an odd run 53 us
// for 4 M cells in four more launches.
template <int PREC, int CL, bool COPY>
__global__ __launch_bounds__(kMaxTile) void k_start(StepArgs A, const ChanInfo *__restrict__ CH,
                                                    const Segment *__restrict__ SEG, int per_wave)
{
    const int lane = threadIdx.x & 63;
    const int wave = (int)blockIdx.x * (kMaxTile / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned long long *const amax_mine =
        A.amax_next + (int64_t)(blockIdx.x & (unsigned)(A.amax_split - 1)) * A.amax_stride;
    unsigned long long acc = 0ull;
    unsigned bad = 0u;
    int c = -1;
    int64_t k = (int64_t)wave * per_wave;
    const int64_t k_end = k + per_wave < A.n_segments ? k + per_wave : A.n_segments;
    while (k < k_end) {
        // the wave's segments of one channel follow one another in memory: one run of cells
        const Segment sg = SEG[k];
        if (c >= 0) {
            const unsigned long long m = wave_max_u64(acc);   // of the channel before
            if (lane == 0 && m != 0ull) flush_max(&amax_mine[c << A.amax_shift], m);
        }
        c = sg.chan;
        int64_t n = sg.n_flags >> 2;
        for (++k; k < k_end && SEG[k].chan == c; ++k) n += SEG[k].n_flags >> 2;
        const double *const z = A.z + sg.cell0;
        double *const hn = A.hn + sg.cell0, *const qn = A.qn + sg.cell0, *const zn = A.zn + sg.cell0;
        acc = speeds_of<PREC, CL>(A.h + sg.cell0, A.q + sg.cell0, (int)n, A.g, closure_of(CH[c]), bad,
                                  [&](int i, double h, double q) {
            if constexpr (COPY) {
                stx(hn, i, h);
                stx(qn, i, q);
                stx(zn, i, ldx(z, i));
            }
        });
        if (COPY && (sg.n_flags & 1u) && lane == 0) A.t_next[c] = A.t_cur[c];
    }
    raise_flag(A.flags, bad);
    merge_max(acc, c, amax_mine, A.amax_shift, true);
}

// cfl_reduce of one channel in one launch: the workgroups' maxima meet in acc[0], and the last of them to
// get there (acc[1] counts) writes the results, the slot that the host checks, and zeroes acc for the next
// call.  Before, clearing, reduction, time step, clearing of the slot and its copy were five launches.
template <int PREC, int CL>
__global__ __launch_bounds__(kCflOneThreads) void k_cfl_one(CflOneArgs A)
{
    __shared__ unsigned long long s_w[kCflOneThreads / 64];
    const int t = (int)threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // even shares in whole rounds of the wave
    const int64_t waves = (int64_t)gridDim.x * (kCflOneThreads / 64);
    const int64_t per = ((A.n + waves - 1) / waves + 63) / 64 * 64;
    const int64_t a = ((int64_t)blockIdx.x * (kCflOneThreads / 64) + wave) * per;
    const int64_t left = A.n - a;
    unsigned bad = 0u;
    unsigned long long acc = 0ull;
    if (left > 0)
        acc = speeds_of<PREC, CL>(A.h + a, A.q + a, (int)(left < per ? left : per), A.g, closure_of(A.ci), bad,
                                  [](int, double, double) {});
    raise_flag(A.flags, bad);
    const unsigned long long m = wave_max_u64(acc);
    if ((t & 63) == 0) s_w[wave] = m;
    __syncthreads();
    if (t != 0) return;
    unsigned long long v = s_w[0];
    for (int w = 1; w < kCflOneThreads / 64; ++w) v = s_w[w] > v ? s_w[w] : v;
    // both atomics return what they replaced, so each has been done when the next begins
    const unsigned long long old = __hip_atomic_fetch_max(&A.acc[0], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(old) : "memory");
    if (__hip_atomic_fetch_add(&A.acc[1], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 != gridDim.x) return;
    const unsigned long long top = __hip_atomic_exchange(&A.acc[0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&A.acc[1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const double amax = __longlong_as_double((long long)top);
    *A.amax = amax;
    *A.dt = A.ci.cfl_dx / amax;
    for (int s = 0; s < kAmaxSplitMax; ++s) A.slot[s * A.slot_stride] = s ? 0ull : top;
}

template <int G, int PREC, int CL>
__global__ __launch_bounds__(256) void k_fluct(FluctArgs A)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned bad = 0u;
    if (e < A.n) {
        double Dm[3], Dp[3];
        edge_fluct<G, PREC, CL>(A.hL[e], A.qL[e], A.zL[e], A.hR[e], A.qR[e], A.zR[e], A.g, closure_of(A.ci),
                                Dm, Dp, bad);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            A.Dm[r * A.n + e] = Dm[r];
            A.Dp[r * A.n + e] = Dp[r];
        }
    }
    raise_flag(A.flags, bad);
}

__global__ __launch_bounds__(256) void k_update(const double *Dm, const double *Dp, const double *dt,
                                                const ChanInfo *ch, double g, int64_t N, double *h,
                                                double *q, double *z)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int64_t E = N + 1;
    const double dti = dt[0];
    const double r = dti * ch->inv_dx;
    const double fric = ch->fric;
    const double h0 = h[i], q0 = q[i];
    double qn = q0 - r * (Dm[E + i + 1] + Dp[E + i]);
    if (fric > 0.0) qn = fma(dti, friction_source(h0, q0, g, fric), qn);
    h[i] = h0 - r * (Dm[i + 1] + Dp[i]);
    q[i] = qn;
    z[i] = z[i] - r * (Dm[2 * E + i + 1] + Dp[2 * E + i]);
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n, unsigned long long v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u32(unsigned int *p, int64_t n, unsigned int v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_copy_u64(unsigned long long *dst, const unsigned long long *src, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// Static device scratch of the allocation-free run (adot_step_noalloc): the ping-pong copy of
// the state and clocks and the rotating CFL slots of a run of at most kNoAllocCells cells in at
// most kNoAllocChannels channels.  Each device the library runs on holds its own copy until the
// process ends.  Host code never passes this name to a kernel: its device address comes from
// hipGetSymbolAddress, once per device (noalloc_scratch below).
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

// ---------------------------------------------------------------------------
static inline unsigned int blocks_for(int64_t n, int bs)
{
    return (unsigned int)((n + bs - 1) / bs);
}

// CFL kernel grid: enough workgroups to fill the chip, few enough that the per-workgroup
// global atomics (serialised on one address per channel) stay cheap.
static inline unsigned int cfl_grid(int64_t n_cells)
{
    const unsigned int full = blocks_for(n_cells, kCflThreads);
    return full < 512u ? full : 512u;
}

template <int PREC>
static hipError_t launch_fluct_prec(const FluctArgs &a, int G, int cl, hipStream_t stream)
{
    const dim3 grid(blocks_for(a.n, 256)), block(256);
#define DSVE_LAUNCH_FLUCT(GG, CC) hipLaunchKernelGGL((k_fluct<GG, PREC, CC>), grid, block, 0, stream, a)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_LAUNCH_FLUCT)
#undef DSVE_LAUNCH_FLUCT
    return hipGetLastError();
}

template <int PREC, bool WIDE>
static hipError_t launch_packed_prec(const StepArgs &a, int G, int cl, int tile, int grid, hipStream_t s)
{
    const size_t lds = sizeof(double) * 6 * (size_t)tile;
#define DSVE_LAUNCH_STEP(GG, CC) hipLaunchKernelGGL((k_step_packed<GG, PREC, CC, WIDE>), dim3(grid), dim3(tile), lds, s, \
                                                   a, a.ch, a.eoff, a.tile_chan, a.amax_cur)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_LAUNCH_STEP)
#undef DSVE_LAUNCH_STEP
    return hipGetLastError();
}

template <int PREC, bool WIDE>
static hipError_t occupancy_query(int G, int cl, int tile, int &n)
{
    const size_t lds = sizeof(double) * 6 * (size_t)tile;
    hipError_t e = hipErrorInvalidValue;
#define DSVE_OCC(GG, CC) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_step_packed<GG, PREC, CC, WIDE>, tile, lds)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_OCC)
#undef DSVE_OCC
    return e;
}

template <bool WIDE>
static hipError_t occupancy_of(int precision, int G, int cl, int tile, int &n)
{
    return precision == PREC_MIXED ? occupancy_query<PREC_MIXED, WIDE>(G, cl, tile, n)
         : precision == PREC_DOT   ? occupancy_query<PREC_DOT, WIDE>(G, cl, tile, n)
                                   : occupancy_query<PREC_FP64, WIDE>(G, cl, tile, n);
}

int packed_blocks_per_cu(int precision, int G, int cl, int tile, int64_t n_edges)
{
    int n = 0;
    const hipError_t e = step_needs_wide_index(n_edges) ? occupancy_of<true>(precision, G, cl, tile, n)
                                                       : occupancy_of<false>(precision, G, cl, tile, n);
    return (e == hipSuccess && n > 0) ? n : 1;
}

template <bool WIDE>
static hipError_t launch_packed_w(const StepArgs &a, int precision, int G, int cl, int tile, int grid,
                                  hipStream_t stream)
{
    if (precision == PREC_FP64) return launch_packed_prec<PREC_FP64, WIDE>(a, G, cl, tile, grid, stream);
    if (precision == PREC_MIXED) return launch_packed_prec<PREC_MIXED, WIDE>(a, G, cl, tile, grid, stream);
    if (precision == PREC_DOT) return launch_packed_prec<PREC_DOT, WIDE>(a, G, cl, tile, grid, stream);
    return hipErrorNotSupported;
}

template <int PREC>
static hipError_t launch_step_prec(const StepArgs &a, int G, int cl, int tile, int grid, hipStream_t s)
{
#define DSVE_LAUNCH_STEP(GG, CC) hipLaunchKernelGGL((k_step<GG, PREC, CC>), dim3(grid), dim3(tile), 0, s, \
                                                   a, a.ch, a.segments, a.amax_cur)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_LAUNCH_STEP)
#undef DSVE_LAUNCH_STEP
    return hipGetLastError();
}

hipError_t launch_step(const StepArgs &a, int precision, int G, int cl, int tile, int grid,
                       hipStream_t stream)
{
    if (tile < 64 || tile > kMaxTile || (tile & 63) || grid < 1) return hipErrorInvalidValue;
    if (a.segments) {
        if ((int64_t)grid * (tile / 64) < a.n_segments) return hipErrorInvalidValue;
        if (precision == PREC_FP64) return launch_step_prec<PREC_FP64>(a, G, cl, tile, grid, stream);
        if (precision == PREC_MIXED) return launch_step_prec<PREC_MIXED>(a, G, cl, tile, grid, stream);
        if (precision == PREC_DOT) return launch_step_prec<PREC_DOT>(a, G, cl, tile, grid, stream);
        return hipErrorNotSupported;
    }
    // workgroup b takes tiles [b lo + min(b, rem), ...), lo + 1 of them for b < rem, else lo
    StepArgs b = a;
    b.tiles_lo = (int32_t)(a.n_tiles / grid);
    b.tiles_rem = (int32_t)(a.n_tiles % grid);
    return step_needs_wide_index(a.n_edges) ? launch_packed_w<true>(b, precision, G, cl, tile, grid, stream)
                                            : launch_packed_w<false>(b, precision, G, cl, tile, grid, stream);
}

template <int PREC>
static hipError_t launch_cfl_prec(const CflArgs &a, int cl, hipStream_t stream)
{
    const dim3 grid(cfl_grid(a.n_cells)), block(kCflThreads);
#define DSVE_LAUNCH_CFL(CC) hipLaunchKernelGGL((k_cfl<PREC, CC>), grid, block, 0, stream, a)
    DSVE_DISPATCH_CL(cl, DSVE_LAUNCH_CFL)
#undef DSVE_LAUNCH_CFL
    return hipGetLastError();
}

hipError_t launch_cfl(const CflArgs &a, int precision, int cl, hipStream_t stream)
{
    if (a.n_cells < 1) return hipErrorInvalidValue;
    if (precision == PREC_FP64) return launch_cfl_prec<PREC_FP64>(a, cl, stream);
    if (precision == PREC_MIXED) return launch_cfl_prec<PREC_MIXED>(a, cl, stream);
    if (precision == PREC_DOT) return launch_cfl_prec<PREC_DOT>(a, cl, stream);
    return hipErrorNotSupported;
}

hipError_t launch_fluct(const FluctArgs &a, int precision, int G, int cl, hipStream_t stream)
{
    if (a.n < 1) return hipSuccess;
    if (precision == PREC_FP64) return launch_fluct_prec<PREC_FP64>(a, G, cl, stream);
    if (precision == PREC_MIXED) return launch_fluct_prec<PREC_MIXED>(a, G, cl, stream);
    if (precision == PREC_DOT) return launch_fluct_prec<PREC_DOT>(a, G, cl, stream);
    return hipErrorNotSupported;
}

hipError_t launch_cell_update(const double *Dm, const double *Dp, const double *dt,
                              const ChanInfo *ch, double g, int64_t N, double *h, double *q,
                              double *z, hipStream_t stream)
{
    if (N < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_update, dim3(blocks_for(N, 256)), dim3(256), 0, stream, Dm, Dp, dt, ch, g,
                       N, h, q, z);
    return hipGetLastError();
}

template <int PREC>
static hipError_t launch_start_prec(const StepArgs &a, int cl, int per_wave, int grid, bool copy, hipStream_t s)
{
#define DSVE_LAUNCH_START(CC)                                                                              \
    if (copy) hipLaunchKernelGGL((k_start<PREC, CC, true>), dim3(grid), dim3(kMaxTile), 0, s, a, a.ch, a.segments, per_wave); \
    else hipLaunchKernelGGL((k_start<PREC, CC, false>), dim3(grid), dim3(kMaxTile), 0, s, a, a.ch, a.segments, per_wave)
    DSVE_DISPATCH_CL(cl, DSVE_LAUNCH_START)
#undef DSVE_LAUNCH_START
    return hipGetLastError();
}

hipError_t launch_start(const StepArgs &a, int precision, int cl, bool copy, hipStream_t stream)
{
    // eight waves to a SIMD at once, each with an even share of the segments
    const int per_wave = (a.n_segments + 8191) / 8192;
    const int waves = (a.n_segments + per_wave - 1) / per_wave, grid = (waves + kMaxTile / 64 - 1) / (kMaxTile / 64);
    if (precision == PREC_FP64) return launch_start_prec<PREC_FP64>(a, cl, per_wave, grid, copy, stream);
    if (precision == PREC_MIXED) return launch_start_prec<PREC_MIXED>(a, cl, per_wave, grid, copy, stream);
    if (precision == PREC_DOT) return launch_start_prec<PREC_DOT>(a, cl, per_wave, grid, copy, stream);
    return hipErrorNotSupported;
}

template <int PREC>
static hipError_t launch_cfl_one_prec(const CflOneArgs &a, int cl, int grid, hipStream_t stream)
{
#define DSVE_LAUNCH_CFL(CC) hipLaunchKernelGGL((k_cfl_one<PREC, CC>), dim3(grid), dim3(kCflOneThreads), 0, stream, a)
    DSVE_DISPATCH_CL(cl, DSVE_LAUNCH_CFL)
#undef DSVE_LAUNCH_CFL
    return hipGetLastError();
}

hipError_t launch_cfl_one(const CflOneArgs &a, int precision, int cl, hipStream_t stream)
{
    if (a.n < 1) return hipErrorInvalidValue;
    // one round of kAhead cells per lane in a workgroup while the chip is not full (two workgroups to a
    // compute unit), then longer shares, whose lengths fit 32 bits to 10^12 cells
    const int64_t round = (int64_t)kCflOneThreads * kAhead;
    const int grid = (int)std::min<int64_t>((a.n + round - 1) / round, 512);
    if (precision == PREC_FP64) return launch_cfl_one_prec<PREC_FP64>(a, cl, grid, stream);
    if (precision == PREC_MIXED) return launch_cfl_one_prec<PREC_MIXED>(a, cl, grid, stream);
    if (precision == PREC_DOT) return launch_cfl_one_prec<PREC_DOT>(a, cl, grid, stream);
    return hipErrorNotSupported;
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s)
{
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u32(unsigned int *p, int64_t n, unsigned int v, hipStream_t s)
{
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

int amax_split_of_kernels() { return kAmaxSplitMax; }

hipError_t launch_copy_u64(unsigned long long *dst, const unsigned long long *src, int64_t n,
                           hipStream_t s)
{
    if (n < 1) return hipSuccess;
    hipLaunchKernelGGL(k_copy_u64, dim3(blocks_for(n, 256)), dim3(256), 0, s, dst, src, n);
    return hipGetLastError();
}

// Device address of `scratch` on the current device, looked up once per device (the device
// must be current; each device holds its own copy of the array at its own address).
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kNoAllocMaxDevices];

hipError_t noalloc_scratch(int device, void **ptr)
{
    *ptr = nullptr;
    if (device < 0 || device >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

}  // namespace dsve
