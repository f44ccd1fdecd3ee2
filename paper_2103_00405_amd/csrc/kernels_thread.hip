// kernels_thread.hip -- thread-per-trajectory mapping for small networks.
//
// One lane owns one trajectory at a time; t, X and each channel's T_k, P_k and
// a_k live in VGPRs, the firing counts n_k and each channel's next draw in LDS,
// the network constants of the wavefront's current item in SGPRs.  The grid is
// persistent: a lane that finishes a trajectory takes the next trajectory of
// the same item, from a range its wavefront reserved, so lanes stay busy despite
// uneven trajectory lengths; a wavefront moves to another item only when all of
// its lanes are idle.
//
// The step is the next reaction random time algorithm (section 4, Table 2)
// in the internal-time form of Eq. 14-16: gaps (P_k - T_k)/a_k, argmin
// (Eq. 25), internal-time advance, jump, and one fresh Exp(1) (Eq. 26).
// The same kernel also runs Gillespie's direct method (section 3, Eq.
// 17-22), the method the paper compares against: total rate a_0 = sum a_k,
// waiting time Exp(1)/a_0 and a search of the running sums for the first to
// reach u a_0, both numbers from one Philox block per firing at counter
// (firing index, 0xFFFFFFFF, trajectory, net).
#include <hip/hip_runtime.h>

#include "internal.h"
#include "rt_device.h"
#include "rt_wave.h"

namespace {

// Where a channel's h_k is found among the products that NT species can make
// (wave-uniform, set once per item).  Up to 4 species every product is made
// once per firing -- 1, X_j, X_i X_j (i < j), X_j^2 - X_j -- and h is entry
// `one` of that list; with 8 species h = e[one] (e[two] - pair) over
// e = (1, X_0 .. X_7).  The entry is picked by register indexing on the uniform
// index: the scalar branches on kind and species that picked it before cost a
// fifth of the kernel's time on a full device (Lotka-Volterra ensemble of 2^20:
// 936 ms with them, 826 ms this way; 750 ms with the model's own propensities
// written out).
struct rt_term {
    int one, two;
    double pair;
    double scale;       // of the rate: 1/2 for a homodimer (its entry is 2 h; exact)
};

template <int NT>
constexpr int term_count() { return NT <= 1 ? 4 : (NT <= 2 ? 8 : 16); }

template <int NT>
__device__ __forceinline__ rt_term channel_term(int kind, int s0, int s1)
{
    rt_term t{0, 0, 0.0, kind == RT_H_PAIR ? 0.5 : 1.0};
    if constexpr (NT <= 4) {
        if (kind == RT_H_ONE) {
            t.one = 1 + s0;
        } else if (kind == RT_H_TWO) {
            const int lo = min(s0, s1), hi = max(s0, s1);
            t.one = 1 + NT + lo * (2 * NT - lo - 1) / 2 + (hi - lo - 1);
        } else if (kind == RT_H_PAIR) {
            t.one = 1 + NT + NT * (NT - 1) / 2 + s0;
        }
    } else {
        t.one = kind == RT_H_ZERO ? 0 : 1 + s0;
        t.two = kind == RT_H_TWO ? 1 + s1 : (kind == RT_H_PAIR ? 1 + s0 : 0);
        t.pair = kind == RT_H_PAIR ? 1.0 : 0.0;
    }
    return t;
}

// a_k = RN(c_k RN(h_k)) of Eq. 1-2 for every channel, X in registers.  Counts
// are below 2^31, so a product of two is exact before its one rounding:
// RN(X_i X_j) is the binary64 product, and a homodimer's 2 RN(h) = RN(X^2 - X)
// one fma (+0 for X = 0 and 1), its factor 1/2 in the rate; no 64-bit integer
// product and one conversion per species.
template <int MT, int NT>
__device__ __forceinline__ void propensities(const rt_term (&q)[MT], const double (&c)[MT],
                                             const int32_t (&X)[NT], double (&a)[MT])
{
    typedef double list_t __attribute__((ext_vector_type(term_count<NT>())));
    double x[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) x[j] = (double)(uint32_t)X[j];
    list_t e;                                              // (the entries past the list are never picked)
    e[0] = 1.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) e[1 + j] = x[j];
    if constexpr (NT <= 4) {
        int at = 1 + NT;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = i + 1; j < NT; ++j) e[at++] = x[i] * x[j];
#pragma unroll
        for (int j = 0; j < NT; ++j) e[at++] = fma(x[j], x[j], -x[j]);
#pragma unroll
        for (int k = 0; k < MT; ++k) a[k] = c[k] * e[q[k].one];
    } else {
#pragma unroll
        for (int k = 0; k < MT; ++k)
            a[k] = c[k] * fma(e[q[k].one], e[q[k].two] - q[k].pair, 0.0);
    }
}

// (m + 1) 2^-53
__device__ __forceinline__ double rt_u53(uint64_t m)
{
    return (fma((double)(uint32_t)(m >> 32), 0x1p32, (double)(uint32_t)m) + 1.0) * 0x1p-53;
}

// The two smallest of MT binary32 values; a NaN makes them equal.
template <int MT>
__device__ __forceinline__ void rt_two_smallest(const float (&v)[MT], float& g1, float& g2)
{
    g1 = v[0];
    g2 = __builtin_inff();
    if constexpr (MT == 3) {
        g1 = fminf(fminf(v[0], v[1]), v[2]);
        g2 = __builtin_amdgcn_fmed3f(v[0], v[1], v[2]);
    } else {
#pragma unroll
        for (int k = 1; k < MT; ++k) {
            g2 = __builtin_amdgcn_fmed3f(g1, g2, v[k]);
            g1 = fminf(g1, v[k]);
        }
    }
}

// Sample points kept in LDS per wavefront.
constexpr int kGridLds = 128;

// Waves per SIMD each instantiation is compiled for: the most at which the
// firing loop's state fits without spilling to scratch (the branches of rare
// events spill up to 88 bytes).
constexpr int thread_min_waves(int MT, int NT, int METHOD, bool SCHED)
{
    if (METHOD == RTSSA_METHOD_DIRECT) return 4;
    // 5 waves up to 3 channels and 2 species (and 2 x 4): 572 ms against 650 for
    // 700000 Lotka-Volterra trajectories at 4, the same for 2^20
    if (!SCHED && ((MT <= 2 && NT <= 4) || (MT == 3 && NT <= 2))) return 5;
    if (!SCHED) return MT <= 4 ? 4 : (MT == 8 && NT == 8 ? 2 : 3);
    // with a schedule each lane also holds its rates in force
    if (MT <= 2 || (MT <= 4 && NT <= 4)) return 4;
    if (MT <= 4 || (MT == 6 && NT <= 4)) return 3;
    return 2;
}

template <int MT, int NT, int METHOD, bool SCHED>
__global__ __launch_bounds__(256, thread_min_waves(MT, NT, METHOD, SCHED)) void rt_thread_kernel(rt_class_dev C)
{
    rt_ws* const ws = C.ws;
    // Issue priority of this kernel's wavefronts over other kernels' sharing a
    // CU (a batch runs class kernels side by side): a small network's class is
    // bound by its longest trajectories, one lane each, so its wavefronts go
    // first; alone on the device every wavefront has the same priority.
    __builtin_amdgcn_s_setprio(3);
    const uint32_t key0 = ws->key0, key1 = ws->key1;
    __shared__ rt_log_lds<4> log_lds;
    const auto sc = log_lds.init();
    // the first points of the item's sample grid, one copy per wavefront: a lane
    // that passes a sample point needs the next one at once, and a global load
    // there stalls its whole wavefront
    __shared__ double sample_points[4][kGridLds];
    double* const sgrid = sample_points[threadIdx.x >> 6];
    __shared__ rt_wave_share wave_shares[4];
    rt_wave_share& share = wave_shares[threadIdx.x >> 6];
    share.clear();
    // firing counts n_k of the lane's trajectory: the count behind the next draw
    // comes from one LDS atomic instead of selects over every channel's register
    __shared__ uint32_t counts[MT][256];
    uint32_t* const cnt = &counts[0][threadIdx.x];
    // with 4 or 8 species the jumps, one row a channel: a lane reads its channel's
    // row (under the channels' masks the jump was MT x NT adds a firing: 7
    // channels, 5 species, 50000 trajectories 5.7 ms, 5.5 ms this way)
    constexpr bool kJumpRows = NT >= 4;
    __shared__ __align__(16) int32_t jump_rows[kJumpRows ? 4 : 1][kJumpRows ? MT * NT : 1];
    int32_t* const jumps = jump_rows[kJumpRows ? threadIdx.x >> 6 : 0];
    // E(k, n_k + 1), the draw channel k's next firing uses
    __shared__ double ahead[METHOD == RTSSA_METHOD_RANDOM_TIME ? MT : 1][256];
    double* const next_draw = &ahead[0][threadIdx.x];

    int item = C.exclusive ? -1 : 0;
    bool first = true;
    for (;;) {
        // ---- the wavefront's next item (uniform)
        if (C.exclusive) {
            unsigned int v = 0;
            if ((threadIdx.x & 63) == 0) v = (unsigned int)atomicAdd(&ws->next_unit, 1ull);
            item = (int)__builtin_amdgcn_readfirstlane((int)__shfl((int)v, 0, 64));
        } else if (!first) {
            item = C.count;
        }
        first = false;
        if (item >= C.count) break;
        share.start_item(C.exclusive != 0);
        // read-only descriptor and network through the constant address space:
        // with a uniform item the loads are scalar and the constants SGPRs
        const rt_cptr<rt_item_dev> it = rt_const(C.items) + item;
        const rt_net_dev net = it->net;
        unsigned long long* const traj_ctr = C.item_next + item;

        // ---- network constants (uniform)
        rt_term terms[MT];
        int nu[MT][NT];
        double c[MT];
#pragma unroll
        for (int k = 0; k < MT; ++k) {
            if (k < net.M) {
                int2 rr = rt_const(net.react)[k];
                terms[k] = channel_term<NT>((int)((uint32_t)rr.x >> 29), rr.x & RT_SPECIES_MASK, rr.y);
                c[k] = terms[k].scale * rt_const(net.c)[k];
            } else {
                terms[k] = channel_term<NT>(RT_H_ZERO, 0, 0);       // dead padding channel
                c[k] = 0.0;
            }
#pragma unroll
            for (int j = 0; j < NT; ++j)
                nu[k][j] = (k < net.M && j < net.N) ? rt_const(net.nu_dense)[k * net.N + j] : 0;
        }
        const int N = net.N, M = net.M;
        // rate schedule of the item (SCHED builds only): breakpoints and rows
        const int32_t sB = SCHED ? net.sched_B : 0;
        const rt_cptr<double> sched_t = rt_const(net.sched_t);
        const rt_cptr<double> sched_c = rt_const(net.sched_c);
        const double t_end = it->t_end;
        const uint32_t net_id = it->net_id, traj_offset = it->traj_offset;
        const bool want_hash = it->seq_hash != nullptr;
        const uint32_t net_k1 = net_id ^ key1;
        // sample rows: X goes straight to memory at each sample point.  A 64-byte
        // line buffer per lane kept the traffic of a launch of 2^20 Lotka-Volterra
        // trajectories at 1.3 GB, where it is 10.1, but a point cost three times the
        // instructions, and 10.1 GB in 0.78 s are 0.3 % of what the card moves.
        // Grids of 10000 points with some 300 firings: 256 trajectories 40.5 ms in
        // the kernel with the buffer, 3.6 without; 40000 trajectories 41.9 and 13.1.
        int32_t* const samples = it->samples;
        const int32_t G = it->G;
        const int64_t ss_n = it->ss_n, ss_g = it->ss_g;
        const bool row2 = NT == 2 && N == 2 && ss_n == 1 &&
                          (((uint64_t)samples >> 2 | (uint64_t)it->ss_r | (uint64_t)ss_g) & 1u) == 0;
        for (int i = (int)(threadIdx.x & 63u); i < kGridLds; i += 64)
            sgrid[i] = i < G ? it->s[i] : __builtin_inf();
        rt_wave_lds_fence();
        auto sample_time = [&](int32_t gg) {
            return gg < kGridLds ? sgrid[gg] : (gg < G ? it->s[gg] : __builtin_inf());
        };
        // counts up to here are safe from any jump's increase
        int32_t up = 0;
#pragma unroll
        for (int k = 0; k < MT; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) up = max(up, nu[k][j]);
        const uint32_t x_safe = 0x7FFFFFFFu - (uint32_t)up;
        if constexpr (kJumpRows) {
            if ((threadIdx.x & 63u) == 0) {
#pragma unroll
                for (int k = 0; k < MT; ++k)
#pragma unroll
                    for (int j = 0; j < NT; ++j) jumps[k * NT + j] = nu[k][j];
            }
            rt_wave_lds_fence();
        }
        bool plain = true;
#pragma unroll
        for (int k = 0; k < MT; ++k) plain = plain && rt_plain_rate(c[k]);

        // ---- trajectory state
        int32_t X[NT];
        double T[MT], Pk[MT], a[MT];
        rt_traj_words tw{0u, 0u};
#pragma unroll
        for (int j = 0; j < NT; ++j) X[j] = 0;
#pragma unroll
        for (int k = 0; k < MT; ++k) { T[k] = 0.0; Pk[k] = 1.0; a[k] = 0.0; }   // (padding: gap +inf)
        double t = 0.0, s_next = __builtin_inf();
        // the earliest of the next sample point, the next rate breakpoint and
        // t_end: a firing past it needs the rare branch (so does every pass of
        // a lane without a trajectory in progress, which holds -1 here)
        double t_stop = -1.0;
        // SCHED: the rates in force for this lane's trajectory, the index of
        // the next breakpoint and its time
        double cl[MT];
        int32_t piece = 0;
        double b_next = __builtin_inf();
#pragma unroll
        for (int k = 0; k < MT; ++k) cl[k] = c[k];
        int32_t g = 0;
        uint32_t fired = 0, tie = kTieNone;
        unsigned long long hash = kFnvOffset;
        uint32_t r = 0;
        int32_t* sp = nullptr;                             // sample row g of trajectory r
        auto write_row = [&](bool invalid) {
            if constexpr (NT == 2) {
                if (row2) {
                    *(int2*)sp = invalid ? make_int2(-1, -1) : make_int2(X[0], X[1]);
                    return;
                }
            }
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (j < N) sp[j * ss_n] = invalid ? -1 : X[j];
        };
        auto refresh = [&]() {
            if constexpr (SCHED) propensities<MT, NT>(terms, cl, X, a);
            else propensities<MT, NT>(terms, c, X, a);
        };

        // Each pass is one firing of every active lane.  Two chains of dependent
        // instructions run side by side in it, so that a wavefront with its SIMD to
        // itself is not bound by their sum: the choice of the firing channel from
        // the state, and the draw that replaces the one the previous firing used
        // (of channel mu_p; a direct-method firing's numbers need no state at all).
        // Side by side they took the ensemble of 2^20 Lotka-Volterra trajectories
        // (a full device, bound by VALU issue) from 826 to 785 ms and a
        // seven-channel network of 50000 from 6.2 to 5.7 ms.
        // Everything up to the one branch for rare events (start or end of a
        // trajectory, a sample point, a close or clamped gap, a logarithm the quick
        // phase left open, an overflow, the firing cap) is straight-line code.
        bool active = (int)(threadIdx.x & 63u) < C.lanes, fresh = true, capped = false;
        uint32_t mu_p = 0u, n_next = 1u;                   // the draw to be made: E(mu_p, n_next)
        double E_now = 0.0, u_now = 0.0;                   // DIRECT: this firing's numbers
        float g_min = plain ? 1e-30f : __builtin_inff();   // smallest gap the binary32 order takes
        // this pass makes a draw again that is counted already: the one before ended
        // a trajectory or a piece (without a schedule, some lane's), and a
        // trajectory's first pass makes E(0, 1)
        bool again = true;
        while (active) {
            double df[MT];
            float gf[MT];
            float g1 = 0.0f;
            unsigned long long fm[MT];                     // lanes in which channel k fires
            uint32_t mu = 0u;
            double d1 = 0.0, t_new = 0.0, E_old = 0.0;
            // ---- the next draw
            auto draw_bits = [&](double& u2) {
                if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                    return rt_block_m53(
                        rt_philox_traj(tw, n_next >> 1, mu_p, net_k1, key0, key1), n_next);
                } else {
                    const rt_u4 w = rt_philox_traj(tw, fired + 1u, 0xFFFFFFFFu, net_k1, key0, key1);
                    u2 = rt_u53((((uint64_t)w.w << 32) | w.z) >> 11);
                    return (((uint64_t)w.y << 32) | w.x) >> 11;
                }
            };
            double E_new, u_new = 0.0;
            const uint64_t m_new = draw_bits(u_new);
            const bool open =
                !rt_neglog_quick((uint32_t)(m_new >> 32), (uint32_t)m_new, sc.tab, E_new);
            // ---- the channel that fires
            // from gf, g1 and df: the firing channel's masks, index, gap and draw
            auto choose = [&]() {
                if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                    double am = a[MT - 1], dm = df[MT - 1];
                    mu = MT - 1;
                    fm[MT - 1] = ~0ull;
#pragma unroll
                    for (int k = MT - 2; k >= 0; --k) {
                        fm[k] = __ballot(gf[k] == g1);
                        const bool f = __builtin_amdgcn_inverse_ballot_w64(fm[k]);
                        am = f ? a[k] : am;
                        dm = f ? df[k] : dm;
                        mu = f ? (uint32_t)k : mu;
                        fm[MT - 1] &= ~fm[k];
                    }
                    d1 = dm * rt_recip(am);
                    E_old = next_draw[mu * 256u];
                } else {
                    // total rate, then the first running sum to reach u2 a_0
                    // (padding channels add +0 and are never reached)
                    double a0 = 0.0;
#pragma unroll
                    for (int k = 0; k < MT; ++k) a0 += a[k];
                    d1 = a0 == 0.0 ? __builtin_inf() : E_now / a0;
                    const double target = u_now * a0;
                    double run = 0.0;
                    unsigned long long left = ~0ull;
                    mu = MT - 1;
#pragma unroll
                    for (int k = 0; k < MT; ++k) {
                        run += a[k];
                        fm[k] = k == MT - 1 ? left : left & __ballot(run >= target);
                        if (k < MT - 1)
                            mu = __builtin_amdgcn_inverse_ballot_w64(fm[k]) ? (uint32_t)k : mu;
                        left &= ~fm[k];
                    }
                }
                t_new = t + d1;
            };
            bool amb = false;
            if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                // The argmin of the gaps (Eq. 25).  Only the smallest gap's value
                // enters the trajectory, so the gaps are first compared in
                // binary32, (P - T) rcp(a) with relative error below 2^-21, and
                // the one exact reciprocal RN(1 / a_mu) is made for the winner:
                // three IEEE divisions per firing (63 issue cycles each) were 15 %
                // of the Lotka-Volterra kernel's issue time.
                // The binary32 order decides when the smallest is above 1e-30 and
                // the second at least 1 + 2^-18 times it (which also excludes
                // near-ties, clamped gaps and values whose binary32 form under- or
                // overflowed); else the exact form below decides.
#pragma unroll
                for (int k = 0; k < MT; ++k) {
                    df[k] = Pk[k] - T[k];
                    gf[k] = (float)df[k] * __builtin_amdgcn_rcpf((float)a[k]);
                }
                float g2;
                rt_two_smallest<MT>(gf, g1, g2);
                amb = !(g1 > g_min) | !(g2 > g1 * (1.0f + 0x1p-18f));
            }
            choose();
            // a jump may leave [0, 2^31 - 1] only upwards (a channel with a_k > 0
            // has its reactants), and only from a count past x_safe
            uint32_t x_top = (uint32_t)X[0];
#pragma unroll
            for (int j = 1; j < NT; ++j) x_top = max(x_top, (uint32_t)X[j]);
            // (NaN, from an absorbed state, is past every time)
            bool late = !(t_new <= t_stop);
            unsigned long long rare = __ballot(x_top > x_safe);
            const unsigned long long ambs = __ballot(amb), opens = __ballot(open);
            if (__builtin_expect((rare | ambs | opens | __ballot(late)) != 0ull, 0)) {
            bool near = false, clamped = false;
            if (opens != 0ull) {
                if (open) {
                    double u2;
                    if (rt_neglog_open(draw_bits(u2), false, sc.sc, E_new) && !again)
                        atomicAdd(&ws->slow_logs, 1ull);
                }
            }
            if (METHOD == RTSSA_METHOD_RANDOM_TIME && ambs != 0ull) {
                if (amb) {
                    // exact gaps: max(0, RN((P - T) RN(1 / a))), +inf for a
                    // frozen channel, lowest k on ties
                    rt_min2 sel{__builtin_inf(), __builtin_inf(), 0};
#pragma unroll
                    for (int k = 0; k < MT; ++k) {
                        const double raw = df[k] * rt_recip(a[k]);
                        rt_min2_push(sel, a[k] == 0.0 ? __builtin_inf() : fmax(raw, 0.0), k);
                    }
                    near = rt_near_tie(sel.d1, sel.d2);
                    g1 = 1.0f;
#pragma unroll
                    for (int k = 0; k < MT; ++k) {
                        gf[k] = sel.k == k ? 1.0f : 2.0f;
                        // (a clamped gap fires at once; when every channel is
                        // frozen the winner's reciprocal gives d1 = NaN)
                        const bool neg = sel.k == k && a[k] != 0.0 && df[k] < 0.0;
                        clamped = clamped || (neg && df[k] * rt_recip(a[k]) < 0.0);
                        df[k] = neg ? 0.0 : df[k];
                    }
                }
                choose();
                late = !(t_new <= t_stop);
                rare |= __ballot(near || clamped);
            }
            // sample points before the event, the commonest of the rare events,
            // apart from the others (idempotent, should the pass be repeated)
            if (s_next < t_new && t_new <= t_end && !(SCHED && b_next < t_end && t_new > b_next)) {
                do {
                    if (samples) {
                        write_row(false);
                        sp += ss_g;
                    }
                    s_next = sample_time(++g);
                } while (s_next < t_new);
                t_stop = fmin(s_next, SCHED ? fmin(b_next, t_end) : t_end);
                late = !(t_new <= t_stop);
            }
            rare |= __ballot(late);
            if (__builtin_expect(rare != 0ull, 0)) {
                const bool live = !fresh && !capped;          // a trajectory is in progress
                const bool absorbed = !(d1 < __builtin_inf());
                // a rate breakpoint before the next firing (and before t_end):
                // Eq. 28 is solved again from there
                const bool brk = SCHED && live && b_next < t_end && (absorbed || t_new > b_next);
                const bool term = !brk && (absorbed || t_new > t_end);
                // the jump, checked exactly: X_j in [0, 2^31 - 1] plus an int32
                // change leaves that range exactly when the 32-bit wrap is negative
                int32_t sign = 0;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    int32_t dl = nu[MT - 1][j];
#pragma unroll
                    for (int k = 0; k < MT - 1; ++k) dl = mu == (uint32_t)k ? nu[k][j] : dl;
                    sign |= (int32_t)((uint32_t)X[j] + (uint32_t)dl);
                }
                const bool ok = sign >= 0;
                const bool event = live && !term && !brk;     // this pass may apply an event
                // Counted once per event: when another lane of the wave stops, this
                // lane may repeat its pass below without applying its event, so
                // the counters are bumped only once the event is known to be
                // applied (or, for a near-tie, when the event ends the trajectory
                // by an overflow, as the oracle counts it); tie is idempotent.
                const bool near_tie = event && near;
                if (near_tie) tie = tie == kTieNone ? fired : tie;
                if (SCHED && brk) {
                    // every internal clock runs to the breakpoint at the old
                    // rates; the propensities take the next piece's rates
                    const double db = b_next - t;
#pragma unroll
                    for (int k = 0; k < MT; ++k) T[k] = fma(a[k], db, T[k]);
                    t = b_next;
#pragma unroll
                    for (int k = 0; k < MT; ++k)
                        cl[k] = k < M ? terms[k].scale * sched_c[piece * M + k] : 0.0;
                    ++piece;
                    b_next = piece < sB ? sched_t[piece] : __builtin_inf();
                    t_stop = fmin(s_next, fmin(b_next, t_end));
                    bool ok_rates = true;
#pragma unroll
                    for (int k = 0; k < MT; ++k) ok_rates = ok_rates && rt_plain_rate(cl[k]);
                    g_min = ok_rates ? 1e-30f : __builtin_inff();
                    refresh();
                }
                const bool stop = !live || term || (!ok && !brk);
                if (near_tie && stop) atomicAdd(&ws->near_ties, 1ull);   // event && !ok
                if (stop && !fresh) {
                    // end of the trajectory
                    const int st = capped ? RTSSA_TRAJ_MAX_FIRINGS
                                          : (absorbed ? RTSSA_TRAJ_ABSORBED
                                                      : (term ? RTSSA_TRAJ_OK : RTSSA_TRAJ_OVERFLOW));
                    const bool good = st == RTSSA_TRAJ_OK || st == RTSSA_TRAJ_ABSORBED;
                    if (samples)
                        for (; g < G; ++g, sp += ss_g) write_row(!good);
                    if (METHOD == RTSSA_METHOD_RANDOM_TIME && good) {
                        const double dt = t_end - t;
#pragma unroll
                        for (int k = 0; k < MT; ++k) T[k] = fma(a[k], dt, T[k]);
                    }
                    if (it->n_out) {
#pragma unroll
                        for (int k = 0; k < MT; ++k) if (k < M) it->n_out[(int64_t)r * M + k] = cnt[k * 256];
                    }
                    if (METHOD == RTSSA_METHOD_RANDOM_TIME && it->T_out) {
#pragma unroll
                        for (int k = 0; k < MT; ++k) if (k < M) it->T_out[(int64_t)r * M + k] = T[k];
                    }
                    if (it->x_final) {
#pragma unroll
                        for (int j = 0; j < NT; ++j) if (j < N) it->x_final[(int64_t)r * N + j] = X[j];
                    }
                    if (it->t_last) it->t_last[r] = t;
                    if (it->status) it->status[r] = (uint8_t)st;
                    if (it->seq_hash) it->seq_hash[r] = hash;
                    if (METHOD == RTSSA_METHOD_RANDOM_TIME && it->tie_step) it->tie_step[r] = tie;
                    share.finished(fired, st);
                }
                if (stop) {
                    // take the next trajectory of this item
                    const int64_t rr = share.take(traj_ctr, it->R);
                    fresh = false;
                    capped = false;
                    active = rr < it->R;
                    if (active) {
                        r = (uint32_t)rr;
                        const uint32_t traj = traj_offset + r;
                        sp = samples ? samples + rr * it->ss_r : nullptr;
                        const int32_t* x0 = it->x0 + (it->x0_per_traj ? rr * N : 0);
#pragma unroll
                        for (int j = 0; j < NT; ++j) X[j] = j < N ? x0[j] : 0;
                        t = 0.0;
                        g = 0;
                        s_next = sample_time(0);
                        fired = 0;
                        tie = kTieNone;
                        hash = kFnvOffset;
                        if constexpr (SCHED) {
                            piece = 0;
                            b_next = sB > 0 ? sched_t[0] : __builtin_inf();
#pragma unroll
                            for (int k = 0; k < MT; ++k) cl[k] = c[k];
                        }
                        t_stop = fmin(s_next, SCHED ? fmin(b_next, t_end) : t_end);
                        refresh();
                        tw = rt_traj_prepare(traj, key0);
#pragma unroll
                        for (int k = 0; k < MT; ++k) cnt[k * 256] = 0u;
                        if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                            g_min = plain ? 1e-30f : __builtin_inff();
                            mu_p = 0u;
                            n_next = 1u;
#pragma unroll
                            for (int k = 0; k < MT; ++k) T[k] = 0.0;
                            // first internal firing times E(k, 0) and next draws
                            // E(k, 1): the two words of one block, a channel at a time
#pragma unroll 1
                            for (int k = 0; k < M; ++k) {
                                const rt_u4 w =
                                    rt_philox_traj(tw, 0u, (uint32_t)k, net_k1, key0, key1);
                                const double E0 = rt_neglog_wave(rt_block_m53(w, 0u), false,
                                                                 &ws->slow_logs, sc);
                                next_draw[k * 256] = rt_neglog_wave(rt_block_m53(w, 1u), false,
                                                                    &ws->slow_logs, sc);
#pragma unroll
                                for (int q = 0; q < MT; ++q) Pk[q] = q == k ? E0 : Pk[q];
                            }
                        } else {
                            const rt_u4 w =
                                rt_philox_traj(tw, 0u, 0xFFFFFFFFu, net_k1, key0, key1);
                            E_now = rt_neglog_wave((((uint64_t)w.y << 32) | w.x) >> 11, false,
                                                   &ws->slow_logs, sc);
                            u_now = rt_u53((((uint64_t)w.w << 32) | w.z) >> 11);
                        }
                    }
                }
                // Started lanes (and lanes past a breakpoint) compute their gaps.  With
                // a schedule the other lanes go on to apply their events: had all
                // of them repeated the pass, a wavefront would make one for every
                // breakpoint of every lane (Lotka-Volterra, 50000 trajectories to
                // t = 5: 100 breakpoints 4.1 ms, 3.7 this way; 2000 breakpoints 19.5
                // and 7.4).  Without one only a trajectory's end comes here, and
                // the masks the rest of the pass would need cost more.
                again = true;
                if constexpr (SCHED) {
                    if (stop || brk) continue;
                } else {
                    if (__ballot(stop) != 0ull) continue;
                }
                // the event is applied below
                if (near_tie) atomicAdd(&ws->near_ties, 1ull);
                if (clamped) atomicAdd(&ws->clamps, 1ull);
            }
            }
            again = false;
            t = t_new;
            ++fired;
            if (want_hash) hash = (hash ^ (unsigned long long)(uint32_t)mu) * kFnvPrime;
            // the fired channel's updates run under its lanes' mask, one
            // instruction each (as selects over the channels the internal times
            // and the jump took six a channel and two a species)
            if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                // internal times advance by a_k Delta (Eq. 15); the fired channel
                // lands exactly on its firing internal time and takes its next
                // draw: the one just made when it fires twice in a row
                next_draw[mu_p * 256u] = E_new;
                const double E = mu == mu_p ? E_new : E_old;
                int32_t dx[NT];
                if constexpr (kJumpRows) {
#pragma unroll
                    for (int j = 0; j < NT; j += 4) {
                        const int4 v = *(const int4*)(jumps + mu * NT + j);
                        dx[j] = v.x; dx[j + 1] = v.y; dx[j + 2] = v.z; dx[j + 3] = v.w;
                    }
                }
#pragma unroll
                for (int k = 0; k < MT; ++k) T[k] = fma(a[k], d1, T[k]);
#pragma unroll
                for (int k = 0; k < MT; ++k)
                    if (__builtin_amdgcn_inverse_ballot_w64(fm[k])) {
                        rt_land(T[k], Pk[k], E);
                        if constexpr (!kJumpRows) {
#pragma unroll
                            for (int j = 0; j < NT; ++j) X[j] += nu[k][j];
                        }
                    }
                if constexpr (kJumpRows) {
#pragma unroll
                    for (int j = 0; j < NT; ++j) X[j] += dx[j];
                }
                mu_p = mu;
                n_next = atomicAdd(&cnt[mu * 256u], 1u) + 2u;
            } else {
                E_now = E_new;
                u_now = u_new;
                atomicAdd(&cnt[mu * 256u], 1u);
#pragma unroll
                for (int k = 0; k < MT; ++k)
                    if (__builtin_amdgcn_inverse_ballot_w64(fm[k])) {
                        asm volatile("");              // (keeps the mask: no selects)
#pragma unroll
                        for (int j = 0; j < NT; ++j) X[j] += nu[k][j];
                    }
            }
            refresh();
            if (__builtin_expect(__ballot(fired >= C.max_firings) != 0ull, 0)) {
                capped = fired >= C.max_firings;
                t_stop = capped ? -1.0 : t_stop;               // (ends without its event)
                s_next = capped ? __builtin_inf() : s_next;
            }
        }
    }
    share.flush(ws);
}

// Prepares one launch: clears the counters of ws and `extra` (item counters),
// sets the Philox key (from key_src when given, so that a captured graph can
// be replayed with new seeds), and for a single run checks its sample grid
// and stores its item descriptor and unit range.  A grid that is not
// non-decreasing within [0, t_end] leaves the run with no work (R = 0 in the
// stored descriptor), marks every trajectory RTSSA_TRAJ_NOT_RUN and sets
// ws->bad_input, so the simulation kernels that follow exit at once and the
// host learns of it without reading the grid itself.
__global__ void rt_setup_kernel(rt_ws* ws, unsigned long long* extra, int64_t n_extra,
                                uint32_t key0, uint32_t key1, const uint32_t* key_src,
                                rt_item_dev item, rt_item_dev* item_dst, int64_t* unit_start,
                                int64_t R)
{
    const int64_t i0 = threadIdx.x + (int64_t)blockIdx.x * blockDim.x;
    const int64_t stride = (int64_t)blockDim.x * gridDim.x;
    for (int64_t i = i0; i < n_extra; i += stride) extra[i] = 0ull;
    bool bad = false;
    if (item_dst && blockIdx.x == 0) {             // uniform over the block
        for (int g = threadIdx.x; g < item.G; g += blockDim.x) {
            const double s = item.s[g];
            bad = bad || !(s >= 0.0 && s <= item.t_end) || (g > 0 && s < item.s[g - 1]);
        }
        bad = __syncthreads_or(bad);
        if (bad && item.status)
            for (int64_t r = threadIdx.x; r < R; r += blockDim.x)
                item.status[r] = (uint8_t)RTSSA_TRAJ_NOT_RUN;
    }
    if (i0 == 0) {
        ws->firings = ws->near_ties = ws->clamps = ws->slow_logs = 0ull;
        for (int q = 0; q < 4; ++q) ws->status_count[q] = 0ull;
        ws->next_unit = 0ull;
        ws->bad_input = bad ? 1ull : 0ull;
        ws->key0 = key_src ? key_src[0] : key0;
        ws->key1 = key_src ? key_src[1] : key1;
        if (item_dst) {
            rt_item_dev it = item;
            if (bad) it.R = 0;
            *item_dst = it;
            unit_start[0] = 0;
            unit_start[1] = bad ? 0 : R;
        }
    }
}

typedef void (*thread_kernel_t)(rt_class_dev);

template <int MT, int NT>
int launch_mn(rt_class_dev C, int* block, int grid, hipStream_t stream, int* grid_used,
              int64_t lanes_wanted, int method, bool sched)
{
    thread_kernel_t kfn = method == RTSSA_METHOD_DIRECT
                              ? rt_thread_kernel<MT, NT, RTSSA_METHOD_DIRECT, false>
                              : (sched ? rt_thread_kernel<MT, NT, RTSSA_METHOD_RANDOM_TIME, true>
                                       : rt_thread_kernel<MT, NT, RTSSA_METHOD_RANDOM_TIME, false>);
    C.lanes = 64;
    int dev = 0, cus = 0;
    if (grid <= 0 || *block <= 0)
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return rt_fail(RTSSA_E_HIP, "device query failed");
    if (*block <= 0) {
        *block = 256;
        if (grid <= 0 && !C.exclusive && lanes_wanted <= 6 * (int64_t)cus) {
            // A small ensemble: single wavefronts of few lanes on three quarters
            // of the CUs.  A firing's latency bounds it, and a wavefront waits
            // for every lane's rare events, so fewer lanes are faster while each
            // wavefront has its CU to itself (Lotka-Volterra from 100, 100 to t = 5,
            // workgroups of 256 full lanes against few lanes: 64 trajectories 1.68
            // and 1.12 ms, 256 1.76 and 1.19, 1000 1.89 and 1.38, 1536 1.93 and
            // 1.47).  The line at 6 a CU is not where few lanes stop being faster:
            // beyond it they measured 1.53 ms for 1.93 at 2000 trajectories, 1.69
            // for 1.95 at 4000, 1.72 for 1.97 at 8000, the same from 16000 on.
            *block = 64;
            C.lanes = (int32_t)std::max<int64_t>(1, (4 * lanes_wanted + 3 * cus - 1) / (3 * cus));
        }
    }
    if (grid <= 0) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, *block, 0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        const int64_t per_block = (int64_t)(*block / 64) * C.lanes;
        const int64_t need = (lanes_wanted + per_block - 1) / per_block;
        const int64_t full = (int64_t)cus * per_cu;
        grid = (int)std::max<int64_t>(1, std::min<int64_t>(need, full));
    }
    if (grid_used) *grid_used = grid;
    hipLaunchKernelGGL(kfn, dim3(grid), dim3(*block), 0, stream, C);
    return hipGetLastError() == hipSuccess ? RTSSA_OK : rt_fail(RTSSA_E_HIP, "thread kernel launch failed");
}

template <int MT>
int launch_m(int N, const rt_class_dev& C, int* block, int grid, hipStream_t stream, int* gu,
             int64_t lanes, int method, bool sched)
{
    if (N <= 1) return launch_mn<MT, 1>(C, block, grid, stream, gu, lanes, method, sched);
    if (N <= 2) return launch_mn<MT, 2>(C, block, grid, stream, gu, lanes, method, sched);
    if (N <= 4) return launch_mn<MT, 4>(C, block, grid, stream, gu, lanes, method, sched);
    return launch_mn<MT, 8>(C, block, grid, stream, gu, lanes, method, sched);
}

}  // namespace

int rt_thread_supported(int M, int N)
{
    return M >= 0 && N >= 0 && M <= RT_THREAD_MAX_M && N <= RT_THREAD_MAX_N;
}

// M and N are the largest of the class (the kernel pads with dead channels
// and absent species); lanes = trajectories wanted in flight; *block <= 0 is
// set to the workgroup size chosen.
int rt_launch_thread(int M, int N, const rt_class_dev& C, int* block, int grid,
                     hipStream_t stream, int* grid_used, int64_t lanes, int method)
{
    const bool sched = C.has_schedule != 0;
    if (sched && method != RTSSA_METHOD_RANDOM_TIME)
        return rt_fail(RTSSA_E_UNSUPPORTED, "rate schedules run with the random-time method");
    if (!rt_thread_supported(M, N))
        return rt_fail(RTSSA_E_UNSUPPORTED, "network too large for the thread mapping");
    if (*block > 256 || *block % 64)
        return rt_fail(RTSSA_E_INVALID, "thread mapping block must be a multiple of 64, <= 256");
    switch (M) {
        case 0:
        case 1: return launch_m<1>(N, C, block, grid, stream, grid_used, lanes, method, sched);
        case 2: return launch_m<2>(N, C, block, grid, stream, grid_used, lanes, method, sched);
        case 3: return launch_m<3>(N, C, block, grid, stream, grid_used, lanes, method, sched);
        case 4: return launch_m<4>(N, C, block, grid, stream, grid_used, lanes, method, sched);
        case 5:
        case 6: return launch_m<6>(N, C, block, grid, stream, grid_used, lanes, method, sched);
        default: return launch_m<8>(N, C, block, grid, stream, grid_used, lanes, method, sched);
    }
}

int rt_launch_setup(rt_ws* ws, unsigned long long* extra, int64_t n_extra, uint32_t key0,
                    uint32_t key1, const uint32_t* key_src, const rt_item_dev* item,
                    rt_item_dev* item_dst, int64_t* unit_start, hipStream_t stream)
{
    rt_item_dev it{};
    if (item) it = *item;
    const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>(64, (n_extra + 255) / 256));
    hipLaunchKernelGGL(rt_setup_kernel, dim3(nb), dim3(256), 0, stream, ws, extra, n_extra, key0,
                       key1, key_src, it, item ? item_dst : nullptr, unit_start,
                       item ? item->R : (int64_t)0);
    return hipGetLastError() == hipSuccess ? RTSSA_OK : rt_fail(RTSSA_E_HIP, "setup launch failed");
}
