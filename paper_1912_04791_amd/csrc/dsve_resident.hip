// dsve_resident.hip -- runs in one launch: k_resident holds a channel of at most 511 cells in one
// workgroup for all steps of a run; k_parts holds each of few channels in one or several.
#include "dsve_device.hpp"

namespace dsve {

// ---------------------------------------------------------------------------
// Maximum over the workgroup (uniform result): wave maxima through LDS.  `s_w` holds one entry
// per wave; consecutive calls are separated by at least one other barrier of the caller.
__device__ __forceinline__ unsigned long long block_max_u64(unsigned long long v, unsigned long long *s_w)
{
    const unsigned long long m = wave_max_u64(v);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = m;
    __syncthreads();
    unsigned long long r = 0ull;
    const int nw = (blockDim.x + 63) >> 6;
    for (int w = 0; w < nw; ++w) r = (s_w[w] > r) ? s_w[w] : r;
    return r;
}

// Channel-resident run: one workgroup of NT threads takes one channel of N < NT cells (thread i
// holds cell i and computes edge i, between cells i-1 and i) through all n steps of the run,
// with the state in registers, the neighbour states and D^- exchanged through LDS, and the
// channel's CFL maximum reduced within the workgroup; then the next channel.  Every value is
// computed as in k_step (same fluctuation, update and speed, same order of operations), so the
// results are bitwise those of the per-step kernels.
//
// Two barriers per step: the first publishes the state, the second the D^- and the waves' CFL maxima
// of that same state, whose speeds are taken beside the fluctuations that need no time step; only the
// update waits for both.
//
// Compiled for 4 waves per SIMD where k_step runs 3 or more: with many channels the barriers leave
// waves waiting, and the fourth makes up for the 36 bytes the FP64 Grass form then spills (2048
// channels of 100-255 cells 8.1 -> 7.4 us a step, 3000 of 150-400 27 -> 20 us).
template <int G, int PREC, int CL, int NT>
__global__ __launch_bounds__(NT, step_min_waves(PREC, CL) < 3 ? step_min_waves(PREC, CL) : 4)
void k_resident(ResidentArgs A)
{
    __shared__ double s_st[3][NT];        // h, q, z of the cells
    __shared__ double s_dm[3][NT + 1];    // D^- of the edges
    __shared__ unsigned long long s_w[NT / 64];
    const int t = threadIdx.x;
    unsigned bad = 0u;
    for (int c = blockIdx.x; c < A.n_channels; c += gridDim.x) {
        const ChanInfo ci = A.ch[c];
        const Closure K = closure_of(ci);
        const int64_t cell0 = A.off[c];
        const int N = (int)(A.off[c + 1] - cell0);
        const bool has_cell = t < N, has_edge = t <= N;
        double h = 0.0, q = 0.0, z = 0.0;
        if (has_cell) {
            h = A.h[cell0 + t];
            q = A.q[cell0 + t];
            z = A.z[cell0 + t];
        }
        double tc = A.t[c];
        for (int n = 0; n < A.n_steps; ++n) {
            if (has_cell) {
                s_st[0][t] = h;
                s_st[1][t] = q;
                s_st[2][t] = z;
            }
            __syncthreads();
            double Dp[3] = {0.0, 0.0, 0.0};
            unsigned long long sp = 0ull;
            if (has_edge) {
                const int il = (t == 0) ? (ci.bcl == BC_PERIODIC ? N - 1 : 0) : t - 1;
                const int ir = (t == N) ? (ci.bcr == BC_PERIODIC ? 0 : N - 1) : t;
                double hL = s_st[0][il], qL = s_st[1][il], zL = s_st[2][il];
                double hR = s_st[0][ir], qR = s_st[1][ir], zR = s_st[2][ir];
                if (t == 0) {
                    hL = ghost_h(ci.bcl, ci.bl, hL);
                    qL = ghost_q(ci.bcl, ci.bl, qL);
                    if (ci.bcl == BC_DIRICHLET) zL = ghost_z(ci.bcl, ci.bl, zL, tc);
                } else if (t == N) {
                    hR = ghost_h(ci.bcr, ci.br, hR);
                    qR = ghost_q(ci.bcr, ci.br, qR);
                    if (ci.bcr == BC_DIRICHLET) zR = ghost_z(ci.bcr, ci.br, zR, tc);
                }
                double Dm[3];
                edge_fluct<G, PREC, CL>(hL, qL, zL, hR, qR, zR, A.g, K, Dm, Dp, bad);
                s_dm[0][t] = Dm[0];
                s_dm[1][t] = Dm[1];
                s_dm[2][t] = Dm[2];
                if (has_cell)
                    sp = (unsigned long long)__double_as_longlong(fabs(cell_speed<PREC, CL>(h, q, A.g, K, bad)));
            }
            const double amax = __longlong_as_double((long long)block_max_u64(sp, s_w));
            const double dt = ci.cfl_dx * rcp_h(amax);
            const double r = dt * ci.inv_dx;
            if (has_cell) {
                // W_i^{n+1} = W_i^n - dt/dx (D^-_{i+1/2} + D^+_{i-1/2}) + dt S(W_i^n) (Sec. 3, Eq. scheme)
                const double hn = h - r * (s_dm[0][t + 1] + Dp[0]);
                double qn = q - r * (s_dm[1][t + 1] + Dp[1]);
                const double zn = z - r * (s_dm[2][t + 1] + Dp[2]);
                if (ci.fric > 0.0) qn = fma(dt, friction_source(h, q, A.g, ci.fric), qn);
                h = hn;
                q = qn;
                z = zn;
            }
            tc += dt;
        }
        if (has_cell) {
            A.h[cell0 + t] = h;
            A.q[cell0 + t] = q;
            A.z[cell0 + t] = z;
        }
        // the maximum of the final state, for the host's check of the run
        __syncthreads();
        unsigned long long sp = 0ull;
        if (has_cell) sp = (unsigned long long)__double_as_longlong(fabs(cell_speed<PREC, CL>(h, q, A.g, K, bad)));
        const unsigned long long amax_bits = block_max_u64(sp, s_w);
        if (t == 0) {
            A.t[c] = tc;
            A.amax[c << A.amax_shift] = amax_bits;
        }
        __syncthreads();   // the next channel reuses the LDS
    }
    raise_flag(A.flags, bad);
}

// ---------------------------------------------------------------------------
// Node terms for each arithmetic, as 64-bit words for the exchange through LDS.
template <int PREC> struct NodeOf;
template <> struct NodeOf<PREC_FP64> {
    using T = Terms64;
    static constexpr int words = 8;
    static __device__ __forceinline__ void pack(const T &v, double w[words])
    {
        w[0] = v.pb, w[1] = v.lam, w[2] = v.p2a, w[3] = v.p2b;
        w[4] = v.s1a, w[5] = v.s1b, w[6] = v.s2a, w[7] = v.s2b;
    }
    static __device__ __forceinline__ T unpack(const double w[words])
    {
        return T{w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]};
    }
};
template <> struct NodeOf<PREC_MIXED> {
    using T = TermsF;
    static constexpr int words = 5;
    static __device__ __forceinline__ double two(float a, float b) { return __hiloint2double(__float_as_int(b), __float_as_int(a)); }
    static __device__ __forceinline__ float lo(double w) { return __int_as_float(__double2loint(w)); }
    static __device__ __forceinline__ float hi(double w) { return __int_as_float(__double2hiint(w)); }
    static __device__ __forceinline__ void pack(const T &v, double w[words])
    {
        w[0] = two(v.wcc, v.A1n), w[1] = two(v.wc, v.A2n), w[2] = two(v.wcP, v.B0), w[3] = two(v.wccP, v.B1);
        w[4] = two(v.B2, 0.0f);
    }
    static __device__ __forceinline__ T unpack(const double w[words])
    {
        return T{lo(w[0]), hi(w[0]), lo(w[1]), hi(w[1]), lo(w[2]), hi(w[2]), lo(w[3]), hi(w[3]), lo(w[4])};
    }
};
template <> struct NodeOf<PREC_DOT> {
    using T = TermsDot;
    static constexpr int words = 6;
    static __device__ __forceinline__ void pack(const T &v, double w[words])
    {
        w[0] = v.a[0], w[1] = v.a[1], w[2] = v.a[2], w[3] = v.aa[0], w[4] = v.aa[1], w[5] = v.aa[2];
    }
    static __device__ __forceinline__ T unpack(const double w[words]) { return T{{w[0], w[1], w[2]}, {w[3], w[4], w[5]}}; }
};

// Node K of the edge.
template <int G, int PREC, int CL>
__device__ __forceinline__ typename NodeOf<PREC>::T node_terms(int k, double hL, double qL, double zL, double hR,
                                                               double qR, double zR, double g, const Closure &K,
                                                               unsigned &bad)
{
    double s = Gauss<G>::s[0], w = Gauss<G>::w[0];
#pragma unroll
    for (int j = 1; j < G; ++j) {
        s = k == j ? Gauss<G>::s[j] : s;
        w = k == j ? Gauss<G>::w[j] : w;
    }
    if constexpr (PREC == PREC_FP64) {
        const Edge64 E = edge64(hL, qL, zL, hR, qR, zR, g);
        const double q = fma(s, E.dq, qL);
        const Node64 n = node_state64<CL>(fma(s, E.dh, hL), q, g, K);
        const bool u = E.one ? E.up : q >= 0.0;
        Terms64 T;
        const bool ok = node_outer<CL>(n, K, u ? 1.0f : -1.0f, w, E.dh, E.dq, E.eta, T);
        if (!ok) T.pb = __longlong_as_double(0x7FF8000000000000ll);
        return T;
    } else if constexpr (PREC == PREC_MIXED) {
        unsigned long long xmax = 0ull;
        const TermsF T = node_mixed<CL>(edgef(hL, qL, zL, hR, qR, zR), s, w, hL, qL, g, K, xmax);
        bad |= arg_flags(xmax, true);
        return T;
    } else {
        const double dW[3] = {hR - hL, qR - qL, zR - zL};
        return node_dot<CL>(fma(s, dW[0], hL), fma(s, dW[1], qL), g, K, dW, bad);
    }
}

// D^- and D^+ of an edge from the terms of its nodes in LDS (t[node][word][slot]), summed in the order
// of fluct64 / fluct_mixed / fluct_dot.
template <int G, int PREC, int CL, int SLOTS>
__device__ __forceinline__ void terms_to_fluct(const double (*t)[NodeOf<PREC>::words][SLOTS], int slot, const Edge64 &E,
                                               double hL, double qL, double zL, double hR, double qR, double zR,
                                               double g, const Closure &K, double Dm[3], double Dp[3], unsigned &bad)
{
    using T = typename NodeOf<PREC>::T;
    T v[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
        double w[NodeOf<PREC>::words];
#pragma unroll
        for (int j = 0; j < NodeOf<PREC>::words; ++j) w[j] = t[k][j][slot];
        v[k] = NodeOf<PREC>::unpack(w);
    }
    if constexpr (PREC == PREC_FP64) {
        bool ok = true;
#pragma unroll
        for (int k = 0; k < G; ++k) ok = ok && v[k].pb == v[k].pb;
        if (__builtin_amdgcn_ballot_w64(!E.one) == 0ull) {
            OuterSums N = first_terms(v[0]);
#pragma unroll
            for (int k = 1; k < G; ++k) add_terms(N, v[k]);
            outer_to_fluct(N, E.up, E.dq, E.gh_eta, Dm, Dp);
        } else {
            TwoSums N;
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const bool u = E.one ? E.up : fma(Gauss<G>::s[k], E.dq, qL) >= 0.0;
                add_terms(N, v[k], u, Gauss<G>::w[k], g * fma(Gauss<G>::s[k], E.dh, hL));
            }
            two_to_fluct(N, E.one, E.up, E.dq, E.gh_eta, E.eta, Dm, Dp);
        }
        if (!ok) fluct64_general<G, CL>(hL, qL, zL, hR, qR, zR, g, K, Dm, Dp, bad);
    } else if constexpr (PREC == PREC_MIXED) {
        float SA[3] = {0.f, 0.f, 0.f}, SB[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < G; ++k) add_terms(SA, SB, v[k]);
        sums_to_fluctf(SA, SB, E.dq, Dm, Dp);
    } else {
        double SA[3] = {0.0, 0.0, 0.0}, SB[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < G; ++k) add_terms(SA, SB, v[k], Gauss<G>::w[k]);
        sums_to_fluct_dot(SA, SB, Dm, Dp);
    }
}

// Mailbox words: 32 bits of data under a 32-bit tag, so a word that carries the tag a reader waits for
// carries its data too, whatever the order in which words become visible.
__device__ __forceinline__ void post(unsigned long long *w, unsigned tag, unsigned v)
{
    __hip_atomic_store(w, ((unsigned long long)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const unsigned long long *w)
{
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits on another workgroup are looked at every 256 looks: true then (most waits end before that).
struct Wait {
    unsigned long long t0 = 0ull, t = 0ull;
    int looks = 0;
    __device__ __forceinline__ bool pause()
    {
        if ((++looks & 255) != 0) return false;
        t = wall_clock64();
        if (t0 == 0ull) t0 = t;
        return true;
    }
    __device__ __forceinline__ bool past(unsigned long long ticks) const { return t - t0 > ticks; }
};
// Why a part stopped before the run's last step (s_stop).
enum { kAllThere = 0, kGone = 1, kAlone = 2, kStalled = 3 };
constexpr unsigned long long kGaveUp = ~0ull;   // in place of a maximum (whose sign bit is clear)

// The arguments of k_parts, read again: what only the paths that are hardly ever taken need would else be
// held in registers through every step (200 steps of 500 cells: 403 -> 387 us).
__device__ __forceinline__ const PartArgs &args_again()
{
    auto *p = (const __attribute__((address_space(4))) PartArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));   // opaque to the compiler
    return *(const PartArgs *)p;
}
// The word that counts the parts of a channel on the device.
__device__ __forceinline__ unsigned long long *there_word(const PartArgs &A, const Part &P)
{
    return A.box + 2 * (int64_t)A.n_parts * (kPartMaxWords + 2 * kPartHaloWords) + (P.id - P.index);
}

// What becomes of part `id` of a channel whose parts have not all shown up in its first step.  Every part
// counts itself once in the low half of `word` before its first post; the high half holds 1 + the part
// that has taken the channel over.  Only while the count is short can a part take over (`late`: it has
// waited long enough), and a part that finds the channel taken leaves, so either every part is on the
// device, and then stays there to the end, or one part does the channel's work and no other waits.
__device__ __forceinline__ int fate_of(unsigned long long *word, unsigned n_parts, unsigned id, bool late)
{
    int fate = kAllThere;
    if ((threadIdx.x & 63) == 0) {
        unsigned long long v = peek(word);
        // (the word changes at most n_parts + 1 times)
        while (late && (v >> 32) == 0ull && (unsigned)v < n_parts) {
            const unsigned long long taken = v | ((unsigned long long)(id + 1u) << 32);
            if (__hip_atomic_compare_exchange_strong(word, &v, taken, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                v = taken;
        }
        if ((v >> 32) != 0ull) fate = (unsigned)(v >> 32) == id + 1u ? kAlone : kGone;
    }
    return __builtin_amdgcn_readfirstlane(fate);
}

// Whether a wait of part P goes on (kAllThere) or how it ends; looked at while the first maxima of a run
// are waited for (first) or after that.
__device__ __forceinline__ int wait_ends(const Wait &wait, bool first)
{
    const PartArgs &A = args_again();
    const Part &P = A.parts[blockIdx.x];
    // the first maxima are there when every part is; from then on all of them stay
    int stop = kAllThere;
    if (first) stop = fate_of(there_word(A, P), (unsigned)P.n_parts, (unsigned)P.id, wait.past(A.wait_ticks));
    return stop == kAllThere && wait.past(A.wait_ticks + A.stall_ticks) ? kStalled : stop;
}

// A whole channel on this workgroup through global memory, all steps from the state in (h, q, z): tiles
// of 64 edges as in k_step, same operations, each wave every kPartThreads / 64-th tile.  For the part
// that took its channel over, which then waits for no other (1800 cells 4.5 us a step, 7040 cells 22,
// against 1.8 and 1.9 of all parts; numerical eigensolver 75 and 240 against 6.6 and 6.7).
template <int G, int PREC, int CL>
__device__ __forceinline__ void run_alone(unsigned &bad)
{
    const PartArgs &A = args_again();
    const int c = A.parts[blockIdx.x].chan;
    const ChanInfo &ci = A.ch[c];
    const Closure K = closure_of(ci);
    double tc = A.t[c];
    constexpr int WAVES = kPartThreads / 64;
    __shared__ unsigned long long s_m[2][WAVES];   // CFL maxima of the waves in even and odd steps
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int N = (int)ci.ncell;                   // (a channel of several parts is short)
    double *src[3] = {A.h + ci.cell0, A.q + ci.cell0, A.z + ci.cell0};
    double *dst[3] = {A.hp + ci.cell0, A.qp + ci.cell0, A.zp + ci.cell0};
    unsigned long long acc = 0ull;
    const auto see = [&](double h, double q) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(cell_speed<PREC, CL>(h, q, A.g, K, bad)));
        acc = b > acc ? b : acc;
    };
    const auto swap_state = [&] {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double *const p = src[k];
            src[k] = dst[k];
            dst[k] = p;
        }
    };
    // an odd run starts from the copy, so that it ends in (h, q, z)
    for (int i = (int)threadIdx.x; i < N; i += kPartThreads) {
        const double h = src[0][i], q = src[1][i];
        see(h, q);
        if (A.n_steps & 1) {
            dst[0][i] = h;
            dst[1][i] = q;
            dst[2][i] = src[2][i];
        }
    }
    if (A.n_steps & 1) swap_state();
    for (int n = 0; n < A.n_steps; ++n) {
        const unsigned long long m = wave_max_u64(acc);
        if (lane == 0) s_m[n & 1][wave] = m;
        __syncthreads();                           // and the state of the step is written
        unsigned long long top = 0ull;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) top = s_m[n & 1][w] > top ? s_m[n & 1][w] : top;
        const double dt = ci.cfl_dx * rcp_h(__longlong_as_double((long long)top));
        const double r = dt * ci.inv_dx;
        acc = 0ull;
        for (int t0 = kSegTile * wave; t0 < N; t0 += kSegTile * WAVES) {
            const int e = t0 + lane < N ? t0 + lane : N;   // lanes past the last edge compute it again
            const int il = e > 0 ? e - 1 : ci.bcl == BC_PERIODIC ? N - 1 : 0;
            const int ir = e < N ? e : ci.bcr == BC_PERIODIC ? 0 : N - 1;
            double hL = src[0][il], qL = src[1][il], zL = src[2][il];
            double hR = src[0][ir], qR = src[1][ir], zR = src[2][ir];
            const double h0 = hL, q0 = qL, z0 = zL;
            if (e == 0) {
                hL = ghost_h(ci.bcl, ci.bl, hL);
                qL = ghost_q(ci.bcl, ci.bl, qL);
                if (ci.bcl == BC_DIRICHLET) zL = ghost_z(ci.bcl, ci.bl, zL, tc);
            } else if (e == N) {
                hR = ghost_h(ci.bcr, ci.br, hR);
                qR = ghost_q(ci.bcr, ci.br, qR);
                if (ci.bcr == BC_DIRICHLET) zR = ghost_z(ci.bcr, ci.br, zR, tc);
            }
            double Dm[3], Dp[3];
            edge_fluct<G, PREC, CL>(hL, qL, zL, hR, qR, zR, A.g, K, Dm, Dp, bad);
            const double p0 = lane_below(Dp[0]), p1 = lane_below(Dp[1]), p2 = lane_below(Dp[2]);
            if (lane > 0 && t0 + lane <= N) {
                // W_i^{n+1} = W_i^n - dt/dx (D^-_{i+1/2} + D^+_{i-1/2}) + dt S(W_i^n) (Sec. 3, Eq. scheme)
                const double hv = h0 - r * (Dm[0] + p0);
                double qv = q0 - r * (Dm[1] + p1);
                const double zv = z0 - r * (Dm[2] + p2);
                if (ci.fric > 0.0) qv = fma(dt, friction_source(h0, q0, A.g, ci.fric), qv);
                dst[0][e - 1] = hv;
                dst[1][e - 1] = qv;
                dst[2][e - 1] = zv;
                see(hv, qv);
            }
        }
        swap_state();
        tc += dt;
    }
    const unsigned long long m = wave_max_u64(acc);
    if (lane == 0 && m != 0ull) atomicMax(&A.amax[c << A.amax_shift], m);
    if (threadIdx.x == 0) A.t[c] = tc;
}

// A run of few channels, all n steps in one launch: one workgroup per part of a channel.
//
// Few channels leave most of the chip idle, and a step takes as long as one wave needs for its chain of
// dependent instructions.  The work of an edge is therefore spread over waves: role k < G takes node k
// of the quadrature, role G the rest: the CFL speeds of its cells, which it keeps in registers, the sum
// of the nodes' terms (in the order of the per-step kernels, so the results are bitwise theirs), the
// exchange of D^+ with the lane above by a DPP move, and the update: lane l of its wave w takes edge
// 63 w + l and updates cell 63 w + l - 1, as in k_step.  Two barriers per step.
//
// A channel longer than one workgroup holds is cut into parts, which take the maximum of their CFL
// maxima through mailboxes once a step (its latency runs beside the nodes), and keep kPartHalo cells of
// their neighbours on either side, of which every step spoils one, refreshed every kPartHalo steps.
//
// Parts wait for one another, so they all have to be on the chip.  Each counts itself in at its start, at
// no cost but an atomic's way there and back beside the first loads; should one be missing when the others
// have waited for it about as long as the run takes on one workgroup (wait_ticks), one of them takes the
// channel over (fate_of, run_alone) and the rest end.  From the first step's maxima on all are there.
//
// Bound by latency: of the 4500 cycles of a step of 17 parts about 2500 pass between the post of a
// part's maximum and the last part's arrival, beside them the nodes; the rest is the speeds' chain
// before it, the update after it, and the barriers.  The waves of role G run at raised priority: they
// share SIMDs with node waves and were held up by them (1.72 -> 1.37 us a step for 100 cells).  One
// channel, per step, against one workgroup per channel or a launch per step: 100 cells 1.6 -> 0.95 us, 500
// cells 2.6 -> 1.7 us, 1800 cells 4.7 -> 1.8 us, 7000 cells 5.2 -> 1.9 us; 100 cells with the numerical
// eigensolver 13.4 -> 5.9 us.  At 128 registers per lane (two workgroups to a compute unit) it spills and
// takes half as long again.
//
// CUT: some channel of the context is cut.  Without, the kernel has nothing of the exchange between parts,
// whose values took registers and scalar moves in every step even of runs that exchange nothing: 100 cells
// 1.23 -> 0.96 us a step, with one node 1.14 -> 0.92, where k_resident took 1.05.
template <int G, int PREC, int CL, bool CUT>
__global__ __launch_bounds__(kPartThreads, 2)
void k_parts(PartArgs A)
{
    constexpr int NW = part_waves(G), NC = part_cells(G), SLOTS = 64 * NW, NWORDS = NodeOf<PREC>::words;
    __shared__ double s_st[3][NC];                // h, q, z of the cells
    __shared__ double s_t[G][NWORDS][SLOTS];      // terms of the nodes
    __shared__ double s_tc;                       // clock of the channel
    __shared__ unsigned long long s_w[NW];        // CFL maxima of the waves
    __shared__ int s_stop;
    const Part P = A.parts[blockIdx.x];
    if (P.n == 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int role = wave / NW, gw = wave - role * NW;
    const int n = P.n, slot = 64 * gw + lane;
    const bool busy = role <= G && 63 * gw < n;       // the wave has edges
    const int e = 63 * gw + lane < n ? 63 * gw + lane : n;
    const int i = e - 1;                              // the cell that role G updates
    const bool mine = role == G && lane > 0 && 63 * gw + lane <= n;
    const bool own = mine && i >= P.own0 && i < P.own1;
    // the channel's record in vector registers (the index is opaque to the compiler): there are enough
    // of them, while as scalars it would be moved in and out of lanes in every step
    int vzero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(vzero));
    const ChanInfo ci = A.ch[P.chan + vzero];
    const Closure K = closure_of(ci);
    const bool cutL = CUT && (P.cut & 1) != 0, cutR = CUT && (P.cut & 2) != 0, many = CUT && P.n_parts > 1;
    const bool ring = ci.bcl == BC_PERIODIC && !many;
    double h = 0.0, q = 0.0, z = 0.0;
    int64_t cell = 0;
    if (mine) {
        cell = P.a + i;                               // (a channel has more cells than a part)
        cell += cell < 0 ? P.ncell : cell >= P.ncell ? -P.ncell : 0;
        cell += P.cell0;
        s_st[0][i] = h = A.h[cell];
        s_st[1][i] = q = A.q[cell];
        s_st[2][i] = z = A.z[cell];
    }
    double tc = A.t[P.chan];
    const int first = P.id - P.index;                 // the channel's first part
    // (the clock has been read when the first barrier is passed: a part that ends writes it)
    if (threadIdx.x == 0) {
        s_tc = tc;
        int stop = kAllThere;
        if (many) {
            if (P.index == A.hold_part && A.hold_step == 0) {
                const unsigned long long t0 = wall_clock64();
                while (wall_clock64() - t0 < 4ull * A.wait_ticks) __builtin_amdgcn_s_sleep(8);
            }
            // here, unless the channel has been taken over (fate_of)
            const unsigned long long was = __hip_atomic_fetch_add(there_word(A, P), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((was >> 32) != 0ull) stop = kGone;
        }
        s_stop = stop;
    }
    unsigned bad = 0u;
    const int left = first + (P.index > 0 ? P.index - 1 : P.n_parts - 1);
    const int right = first + (P.index + 1 < P.n_parts ? P.index + 1 : 0);
    // mailboxes of the maxima: this wave's word, and up to kLooks words per lane that it reads
    constexpr int kLooks = kMaxParts * 2 * NW / 64;
    const int words = P.n_parts * 2 * NW, looks = (words + 63) / 64;
    unsigned long long *my_word = A.box + (int64_t)P.id * kPartMaxWords + 2 * gw + lane;
    unsigned long long *look[kLooks];
#pragma unroll
    for (int k = 0; k < kLooks; ++k) {
        const int j = 64 * k + lane < words ? 64 * k + lane : lane & 1;
        look[k] = A.box + (int64_t)(first + j / (2 * NW)) * kPartMaxWords + j % (2 * NW);
        asm volatile("" : "+v"(look[k]));   // kept, not formed again from the arguments in every step
    }
    asm volatile("" : "+v"(my_word));
    // and of the cells next to the cuts: where this lane's cell goes on either side, and where it comes from
    unsigned long long *halo_out[2], *halo_in;
    {
        unsigned long long *const box_halo = A.box + 2 * (int64_t)A.n_parts * kPartMaxWords;
        const bool lo_side = mine && cutL && i < P.own0, hi_side = mine && cutR && i >= P.own1;
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const int at = side ? i - (P.own1 - kPartHalo) : i - P.own0;
            halo_out[side] = box_halo + ((int64_t)P.id * 2 + side) * kPartHaloWords + at * 6;
            asm volatile("" : "+v"(halo_out[side]));
        }
        // the left neighbour's cells next to its right cut, the right one's next to its left
        const int64_t from = lo_side ? ((int64_t)left * 2 + 1) * kPartHaloWords : (int64_t)right * 2 * kPartHaloWords;
        halo_in = box_halo + from + (lo_side ? i : hi_side ? i - P.own1 : 0) * 6;
        asm volatile("" : "+v"(halo_in));
    }
    // The waves of role G are what a step waits for: they go first where waves share a SIMD.
    if (role == G) __builtin_amdgcn_s_setprio(3);
    int v0 = 0, v1 = n;                               // cells whose state is that of the step
    const int n_steps = many && P.index == A.hold_part && A.hold_step > 0 && A.hold_step < A.n_steps ? A.hold_step : A.n_steps;
    int step = 0;
    for (; step < n_steps; ++step) {
        __syncthreads();
        if (many && s_stop) break;
        const int w0 = v0 + (cutL ? 1 : 0), w1 = v1 - (cutR ? 1 : 0);   // cells of the next state
        const bool needed = e >= w0 && e <= w1;                        // faces of those
        double hL = 0.0, qL = 0.0, zL = 0.0, hR = 0.0, qR = 0.0, zR = 0.0, fs = 0.0;
        Edge64 E;
        unsigned edge_bad = 0u;
        const unsigned tag = (unsigned)step + 1u;
        const int64_t parity = (int64_t)(step & 1) * A.n_parts * kPartMaxWords;
        if (role == G) {
            // CFL speeds of the part's own cells
            unsigned long long sp = 0ull;
            if (own) sp = (unsigned long long)__double_as_longlong(fabs(cell_speed<PREC, CL>(h, q, A.g, K, bad)));
            const unsigned long long m = wave_max_u64(sp);
            if (!many) {
                if (lane == 0) s_w[gw] = m;
            } else if (lane < 2) {
                post(my_word + parity, tag, lane ? (unsigned)m : (unsigned)(m >> 32));
            }
        }
        if (busy) {
            const int il = e > 0 ? e - 1 : ring ? n - 1 : 0, ir = e < n ? e : ring ? 0 : n - 1;
            hL = s_st[0][il];
            qL = s_st[1][il];
            zL = s_st[2][il];
            hR = s_st[0][ir];
            qR = s_st[1][ir];
            zR = s_st[2][ir];
            if (e == 0 && !cutL) {
                hL = ghost_h(ci.bcl, ci.bl, hL);
                qL = ghost_q(ci.bcl, ci.bl, qL);
                if (ci.bcl == BC_DIRICHLET) zL = ghost_z(ci.bcl, ci.bl, zL, s_tc);
            } else if (e == n && !cutR) {
                hR = ghost_h(ci.bcr, ci.br, hR);
                qR = ghost_q(ci.bcr, ci.br, qR);
                if (ci.bcr == BC_DIRICHLET) zR = ghost_z(ci.bcr, ci.br, zR, s_tc);
            }
            if (role < G) {
                const typename NodeOf<PREC>::T v = node_terms<G, PREC, CL>(role, hL, qL, zL, hR, qR, zR, A.g, K, edge_bad);
                double w[NWORDS];
                NodeOf<PREC>::pack(v, w);
#pragma unroll
                for (int j = 0; j < NWORDS; ++j) s_t[role][j][slot] = w[j];
            } else {
                E = edge64(hL, qL, zL, hR, qR, zR, A.g);
                if (ci.fric > 0.0) fs = friction_source(h, q, A.g, ci.fric);
            }
        }
        __syncthreads();
        if (role == G) {
            // the channel's CFL maximum: of this workgroup's waves, or (below) of all parts
            unsigned long long amax = 0ull;
            double dt = 0.0;
            if (!many) {
                amax = s_w[0];
#pragma unroll
                for (int j = 1; j < NW; ++j)
                    if (63 * j < n) amax = s_w[j] > amax ? s_w[j] : amax;
                dt = ci.cfl_dx * rcp_h(__longlong_as_double((long long)amax));
            }
            double Dm[3] = {0.0, 0.0, 0.0}, Dp[3] = {0.0, 0.0, 0.0};
            if (busy) terms_to_fluct<G, PREC, CL, SLOTS>(s_t, slot, E, hL, qL, zL, hR, qR, zR, A.g, K, Dm, Dp, edge_bad);
            const double s0 = Dm[0] + lane_below(Dp[0]), s1 = Dm[1] + lane_below(Dp[1]), s2 = Dm[2] + lane_below(Dp[2]);
            if (many) {
                Wait wait;
                int stop = kAllThere;
                unsigned long long v[kLooks];
                for (;;) {
                    bool ready = true;
#pragma unroll
                    for (int k = 0; k < kLooks; ++k)
                        if (k < looks) v[k] = peek(look[k] + parity);
#pragma unroll
                    for (int k = 0; k < kLooks; ++k)
                        if (k < looks) ready = ready && (unsigned)(v[k] >> 32) == tag;
                    if (__builtin_amdgcn_ballot_w64(!ready) == 0ull) break;
                    if (__builtin_expect(!wait.pause(), 1)) continue;
                    stop = wait_ends(wait, step == 0);
                    if (stop != kAllThere) {
                        amax = kGaveUp;
                        break;
                    }
                }
                if (amax == kGaveUp) {
                    if (lane == 0) s_stop = stop;
                    if (stop == kStalled) bad |= kFlagTimeout;
                } else {
                    // even lanes read high halves, odd lanes the low halves below them
#pragma unroll
                    for (int k = 0; k < kLooks; ++k)
                        if (k < looks) {
                            const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v[k], 0xB1, 0xf, 0xf, true);
                            const unsigned long long f = (lane & 1) ? 0ull : ((v[k] << 32) | lo);
                            amax = f > amax ? f : amax;
                        }
                    amax = wave_max_u64(amax);
                }
                dt = ci.cfl_dx * rcp_h(__longlong_as_double((long long)amax));
            }
            const double r = dt * ci.inv_dx;
            if (mine && i >= w0 && i < w1 && amax != kGaveUp) {
                // W_i^{n+1} = W_i^n - dt/dx (D^-_{i+1/2} + D^+_{i-1/2}) + dt S(W_i^n) (Sec. 3, Eq. scheme)
                h = h - r * s0;
                q = q - r * s1;
                z = z - r * s2;
                if (ci.fric > 0.0) q = fma(dt, fs, q);
                s_st[0][i] = h;
                s_st[1][i] = q;
                s_st[2][i] = z;
            }
            tc += dt;
            if (threadIdx.x == 64 * NW * G) s_tc = tc;
        }
        if (needed) bad |= edge_bad;
        v0 = w0;
        v1 = w1;
        if (many && role == G && (step + 1) % kPartHalo == 0 && step + 1 < n_steps) {
            // own cells next to a cut go out, the neighbours' come in
            const int64_t hb = (int64_t)(((step + 1) / kPartHalo) & 1) * A.n_parts * 2 * kPartHaloWords;
            const double v[3] = {h, q, z};
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int at = side ? i - (P.own1 - kPartHalo) : i - P.own0;
                if (own && (side ? cutR : cutL) && at >= 0 && at < kPartHalo) {
                    unsigned long long *const w = halo_out[side] + hb;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const unsigned long long x = (unsigned long long)__double_as_longlong(v[k]);
                        post(w + 2 * k, tag, (unsigned)(x >> 32));
                        post(w + 2 * k + 1, tag, (unsigned)x);
                    }
                }
            }
            const bool lo_side = mine && cutL && i < P.own0, hi_side = mine && cutR && i >= P.own1;
            if (__builtin_amdgcn_ballot_w64(lo_side || hi_side) != 0ull) {
                const unsigned long long *const w = halo_in + hb;
                unsigned long long x[6];
                Wait wait;
                bool got = true;
                for (;;) {
                    bool ready = true;
#pragma unroll
                    for (int k = 0; k < 6; ++k) x[k] = peek(w + k);
#pragma unroll
                    for (int k = 0; k < 6; ++k) ready = ready && (unsigned)(x[k] >> 32) == tag;
                    if (__builtin_amdgcn_ballot_w64((lo_side || hi_side) && !ready) == 0ull) break;
                    if (wait.pause() && wait_ends(wait, false) != kAllThere) {
                        got = false;
                        break;
                    }
                }
                if (!got) {
                    // (read after the next barrier)
                    if (lane == 0) s_stop = kStalled;
                    bad |= kFlagTimeout;
                } else if (lo_side || hi_side) {
                    s_st[0][i] = h = __longlong_as_double((long long)((x[0] << 32) | (unsigned)x[1]));
                    s_st[1][i] = q = __longlong_as_double((long long)((x[2] << 32) | (unsigned)x[3]));
                    s_st[2][i] = z = __longlong_as_double((long long)((x[4] << 32) | (unsigned)x[5]));
                }
            }
        }
        if (many && (step + 1) % kPartHalo == 0) {
            v0 = 0;
            v1 = n;
        }
    }
    const PartArgs &B = args_again();
    const Part &PB = B.parts[blockIdx.x];
    if (many) {
        // nothing of a run that did not come to its end is written: the part that finds another missing
        // in a step leaves, and so do all others in that step or the next
        __syncthreads();
        const int stop = s_stop;
        if constexpr (CUT)
            if (stop == kAlone) run_alone<G, PREC, CL>(bad);
        if (stop != kAllThere || step < B.n_steps) {
            raise_flag(B.flags, bad);
            return;
        }
    }
    unsigned long long sp = 0ull;
    if (own) {
        B.h[cell] = h;
        B.q[cell] = q;
        B.z[cell] = z;
        sp = (unsigned long long)__double_as_longlong(fabs(cell_speed<PREC, CL>(h, q, B.g, K, bad)));
    }
    // the maximum of the final state, for the host's check of the run
    if (role == G) {
        const unsigned long long m = wave_max_u64(sp);
        if (lane == 0 && m != 0ull) atomicMax(&B.amax[PB.chan << B.amax_shift], m);
    }
    if (PB.index == 0 && threadIdx.x == 64 * NW * G) B.t[PB.chan] = tc;
    raise_flag(B.flags, bad);
}

template <int PREC, int NT>
static hipError_t launch_resident_prec(const ResidentArgs &a, int G, int cl, int grid, hipStream_t s)
{
#define DSVE_LAUNCH_RES(GG, CC) hipLaunchKernelGGL((k_resident<GG, PREC, CC, NT>), dim3(grid), dim3(NT), 0, s, a)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_LAUNCH_RES)
#undef DSVE_LAUNCH_RES
    return hipGetLastError();
}

template <int NT>
static hipError_t launch_resident_nt(const ResidentArgs &a, int precision, int G, int cl, int grid,
                                     hipStream_t stream)
{
    if (precision == PREC_FP64) return launch_resident_prec<PREC_FP64, NT>(a, G, cl, grid, stream);
    if (precision == PREC_MIXED) return launch_resident_prec<PREC_MIXED, NT>(a, G, cl, grid, stream);
    if (precision == PREC_DOT) return launch_resident_prec<PREC_DOT, NT>(a, G, cl, grid, stream);
    return hipErrorNotSupported;
}

hipError_t launch_resident(const ResidentArgs &a, int precision, int G, int cl, int threads, int grid,
                           hipStream_t stream)
{
    if (grid < 1 || a.n_channels < 1 || a.n_steps < 1) return hipErrorInvalidValue;
    if (threads == 256) return launch_resident_nt<256>(a, precision, G, cl, grid, stream);
    if (threads == 512) return launch_resident_nt<512>(a, precision, G, cl, grid, stream);
    return hipErrorInvalidValue;
}

template <int PREC, bool CUT>
static hipError_t launch_parts_prec(const PartArgs &a, int G, int cl, int grid, hipStream_t s)
{
#define DSVE_LAUNCH_PARTS(GG, CC) hipLaunchKernelGGL((k_parts<GG, PREC, CC, CUT>), dim3(grid), dim3(kPartThreads), 0, s, a)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_LAUNCH_PARTS)
#undef DSVE_LAUNCH_PARTS
    return hipGetLastError();
}

template <int PREC>
static hipError_t parts_occupancy(int G, int cl, int &n)
{
    hipError_t e = hipErrorInvalidValue;
#define DSVE_OCC(GG, CC) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_parts<GG, PREC, CC, true>, kPartThreads, 0)
    DSVE_DISPATCH_G_CL(G, cl, DSVE_OCC)
#undef DSVE_OCC
    return e;
}

int parts_per_cu(int precision, int G, int cl)
{
    int n = 0;
    const hipError_t e = precision == PREC_MIXED ? parts_occupancy<PREC_MIXED>(G, cl, n)
                       : precision == PREC_DOT   ? parts_occupancy<PREC_DOT>(G, cl, n)
                                                 : parts_occupancy<PREC_FP64>(G, cl, n);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess && n > 0 ? n : 0;
}

template <bool CUT>
static hipError_t launch_parts_cut(const PartArgs &a, int precision, int G, int cl, int grid, hipStream_t stream)
{
    if (precision == PREC_FP64) return launch_parts_prec<PREC_FP64, CUT>(a, G, cl, grid, stream);
    if (precision == PREC_MIXED) return launch_parts_prec<PREC_MIXED, CUT>(a, G, cl, grid, stream);
    if (precision == PREC_DOT) return launch_parts_prec<PREC_DOT, CUT>(a, G, cl, grid, stream);
    return hipErrorNotSupported;
}

hipError_t launch_parts(const PartArgs &a, int precision, int G, int cl, int grid, hipStream_t stream)
{
    if (grid < 1 || a.n_steps < 1) return hipErrorInvalidValue;
    return a.n_channels < a.n_parts ? launch_parts_cut<true>(a, precision, G, cl, grid, stream)
                                    : launch_parts_cut<false>(a, precision, G, cl, grid, stream);
}

}  // namespace dsve
