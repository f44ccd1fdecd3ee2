// kernels_subwave.hip -- L lanes per trajectory (L = 4 .. 64), 64 / L
// trajectories per wavefront, for mid-size networks.
//
// Channel k of a trajectory belongs to lane k mod L of its group, slot k / L;
// T_k and P_k live in that lane's VGPRs (slots past the network's M are frozen
// channels that never win).  LDS holds, per wavefront and slot, a_k, a
// binary32 1 / a_k, the channel's next draw E(k, n_k + 1) and n_k, at
// [slot][lane] (no bank conflicts), and each group's species counts X.  The
// groups of a wavefront advance in lockstep, one firing per pass, each with its
// own trajectory.  There are no workgroup barriers: a group lives inside one
// wavefront, whose LDS accesses complete in program order.
//
// One firing (section 4, Table 2, in the internal-time form of Eq. 14-16):
//   selection  the gaps (P_k - T_k) / a_k in binary32, the channel index in
//              their low bits, so that one 32-bit minimum per lane exchange
//              finds both (Eq. 25); the winner's exact gap from one reciprocal.
//              Where the second smallest is within 2^-12 of the smallest, or a
//              value is not a plain positive number, the exact binary64
//              selection with second minimum runs instead;
//   rows       mu's fixed-stride rows in one round trip: its jump and the
//              records of the channels D(mu) (Gibson & Bruck's dependency
//              graph, cited in section 5), each with its reactants, rate and
//              the reactants' changes under v_mu; while they load, waiting
//              draws are made, one slot per lane, when 16 lanes have one or a
//              group's mu fires before its draw is there;
//   event      T_k += a_k Delta, T_mu = P_mu, P_mu += E (Eq. 15, 26), new a_k
//              of D(mu) by the lanes holding its records, X + v_mu.
// Measured (45 channels, 20000 trajectories, with the score gradient: 9.8 ms
// before, 4.0 ms; 301 channels, 4000 trajectories: 44.8, 14.5 ms -- 20.4 at 6
// slots and 12 wavefronts a CU, where 5 slots leave room for all 4000) against
// the kernel this replaced, which kept a_k and 1 / a_k in registers, refreshed them
// one stale slot at a time from the network tables, reduced (gap, second gap,
// channel) in binary64 and made each draw in one lane a group.
//
// Work units are trajectories of the class's items, taken from a device
// counter by one lane per group; every rare event (start or end of a
// trajectory, a sample point, a near-tie, a clamped gap, an overflow, the
// firing cap) is handled in a branch entered only when some group needs it.
// With piecewise-constant rates (SCHED, Eq. 28), a rate breakpoint passed by
// a group's next firing is one more such event: the group's clocks run to the
// breakpoint at the old rates, every propensity takes the new ones, and the
// pass is repeated.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "rt_device.h"
#include "rt_wave.h"

namespace {

// Wavefronts of a workgroup, which share one 6 KiB logarithm table, at most.
constexpr int kWaves = 4;

// Draws are made once this many lanes of a wavefront wait for one.
constexpr int kDrawLanes = 16;

// Waves per SIMD the register allocation must allow (no more fit in LDS: 10 a CU
// at 8 slots, 12 at 6, 16 below).
constexpr int subwave_min_waves(int S) { return S <= 5 ? 4 : 3; }

// LDS bytes of one wavefront: per slot and lane a_k, the next draw, 1 / a_k
// and n_k; then X of each group.
constexpr size_t wave_lds_bytes(int L, int S, int NP)
{
    return (size_t)S * 64 * 24 + (size_t)(64 / L) * NP * 4;
}

template <int L, int S, bool SCHED>
__global__ __launch_bounds__(64 * kWaves, subwave_min_waves(S)) void rt_subwave_kernel(rt_class_dev C)
{
    constexpr int G = 64 / L;                              // groups of a wavefront
    constexpr int LOG2L = __builtin_ctz(L);
    constexpr int32_t kKey = 8 * L - 1;                    // channel bits of a selection key
    constexpr unsigned long long kGroupBits = L == 64 ? ~0ull : ((1ull << L) - 1ull);
    rt_ws* const ws = C.ws;
    // Issue priority over other kernels' wavefronts sharing a CU (batches):
    // below the thread mapping's, above the lazy and workgroup kernels'.
    __builtin_amdgcn_s_setprio(2);
    const uint32_t key0 = ws->key0, key1 = ws->key1;
    const int tid = threadIdx.x, lane = tid & 63, li = lane % L, gbase = lane - li;
    const unsigned long long gmask = kGroupBits << gbase;
    extern __shared__ __align__(16) char dyn_lds[];
    __shared__ rt_log_lds<kWaves> log_lds;
    const auto sc = log_lds.init();
    __shared__ rt_wave_share wave_shares[kWaves];
    rt_wave_share& share = wave_shares[tid >> 6];
    share.clear();
    share.start_item(false);
    const int NP = (C.max_N + 3) & ~3;
    // this lane's slots: entry s 64 of each array
    double* const la = (double*)(dyn_lds + (tid >> 6) * wave_lds_bytes(L, S, NP)) + lane;
    double* const le = la + S * 64;
    float* const linv = (float*)(le - lane + S * 64) + lane;
    uint32_t* const lnk = (uint32_t*)(linv + S * 64);
    int32_t* const X = (int32_t*)(lnk - lane + S * 64) + (lane / L) * NP;
    // offset from this lane's entries to channel k's of its group
    auto at = [&](int k) { return ((k >> LOG2L) << 6) + (k & (L - 1)) - li; };
    const rt_cptr<int64_t> unit_start = rt_const(C.unit_start);
    const int64_t total = unit_start[C.count];

    // channel state of this lane's slots
    double T[S], P[S];
#pragma unroll
    for (int s = 0; s < S; ++s) { T[s] = 0.0; P[s] = __builtin_inf(); }
    // trajectory context (identical in every lane of the group)
    rt_cptr<rt_item_dev> it = rt_const(C.items);
    int M = 0, N = 0;
    int64_t r = 0;
    uint32_t traj = 0, net_id = 0, fired = 0, tie = kTieNone;
    double t = 0.0, t_end = 0.0, s_next = 0.0;
    int32_t g = 0;
    unsigned long long hash = kFnvOffset;
    bool active = true, fresh = true, capped = false;
    uint32_t waiting = 0u;                                 // slots whose next draw is not made yet
    float g_min = 1e-30f;                                  // smallest gap the binary32 order takes
    // rate schedule: breakpoints passed, and the next one
    int32_t piece = 0;
    double b_next = __builtin_inf();
    // a fresh group passes through its first pass with defined values
#pragma unroll
    for (int s = 0; s < S; ++s) { la[s * 64] = 0.0; linv[s * 64] = __builtin_inff(); }
    rt_wave_lds_fence();

    while (active) {
        const rt_cptr<rt_net_dev> net = &it->net;
        // ---- selection
        double df[S];
        int32_t k1 = 0x7FFFFFFF, k2 = 0x7FFFFFFF;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            df[s] = P[s] - T[s];
            const float gap = (float)df[s] * linv[s * 64];
            const int32_t key = (int32_t)rt_and_or(__float_as_uint(gap), (uint32_t)~kKey,
                                                   (uint32_t)(s * L + li));
            k2 = rt_med3_i32(k1, k2, key);
            k1 = min(k1, key);
        }
        const int32_t kbest = rt_group_min_i32<L>(k1);
        int mu = kbest & kKey;
        // rare: the second smallest is close (a lane's candidate: its smallest,
        // or its second where it owns mu), or the smallest is no plain number
        const float gap1 = __uint_as_float((uint32_t)(kbest & ~kKey));
        const int32_t reach = __float_as_int(gap1 * (1.0f + 0x1p-12f)) | kKey;
        const bool amb = !(gap1 > g_min) | ((k1 == kbest ? k2 : k1) <= reach);
        // the winner's exact gap, from its owner lane's P - T
        double dm = df[0];
#pragma unroll
        for (int s = 1; s < S; ++s) dm = (mu >> LOG2L) == s ? df[s] : dm;
        const double a_mu = la[at(mu)];
        dm = __shfl(dm, gbase + (mu & (L - 1)), 64);
        double d1 = dm * rt_recip(a_mu);
        bool near = false, clamped = false;
        const unsigned long long ambs = __ballot(amb);
        if (__builtin_expect(ambs != 0ull, 0)) {
            if ((ambs & gmask) != 0ull) {
                // the exact form: max(0, RN((P - T) RN(1 / a))), +inf for a
                // frozen channel, lowest k on ties, second minimum
                rt_min2 loc = rt_min2_empty();
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const double a = la[s * 64];
                    const double raw = df[s] * rt_recip(a);
                    rt_min2_push(loc, a == 0.0 ? __builtin_inf() : fmax(raw, 0.0), s);
                }
                loc = rt_min2_slot_to_channel(loc, li, LOG2L);
                loc = rt_min2_allreduce<L>(loc);
                d1 = loc.d1;
                mu = loc.k == 0x7FFFFFFF ? 0 : loc.k;
                near = rt_near_tie(loc.d1, loc.d2);
                // a zero gap: was it clamped from a negative raw gap?
                if (d1 == 0.0 && li == (mu & (L - 1))) {
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        if ((mu >> LOG2L) == s) clamped = df[s] * rt_recip(la[s * 64]) < 0.0;
                }
            }
        }
        const double t_new = t + d1;
        const bool own = li == (mu & (L - 1));
        const int sm = mu >> LOG2L;
        // ---- mu's rows, one round trip: its jump (lane li < nu_stride: entry
        // li) and the first records (lane li: record li, then li + L); a mu
        // that does not fire (or is none) has rows as well
        constexpr int kR = G > 1 ? 2 : 1;
        const int mr = M > 0 ? min(mu, M - 1) : 0;
        const int nu_stride = net->nu_stride;
        const int n_other = rt_const(net->touch)[mr * 64];
        const int2 nv = rt_const(net->nu_fixed)[mr * nu_stride + min(li, nu_stride - 1)];
        int4 rec[kR];
        double rc[kR];
        int2 rd[kR];
#pragma unroll
        for (int q = 0; q < kR; ++q) {
            rec[q] = rt_const(net->grow)[mr * 64 + li + q * L];
            rc[q] = rt_const(net->growc)[mr * 64 + li + q * L];
            rd[q] = rt_const(net->gdel)[mr * 64 + li + q * L];
        }
        const bool live = !fresh && !capped;
        // ---- draws while the rows load
        const bool need = live && own && ((waiting >> sm) & 1u);
        const unsigned long long waiters = __ballot(waiting != 0u);
        if (__ballot(need) != 0ull || __popcll(waiters) >= kDrawLanes) {
            if (waiting != 0u) {
                const int s1 = need ? sm : __builtin_ctz(waiting);
                const uint32_t n1 = lnk[s1 * 64] + 1u;
                bool acc;
                const double E = rt_exp1_wave(key0, key1, traj, net_id, (uint32_t)(s1 * L + li), n1,
                                              &ws->slow_logs, sc, &acc);
                le[s1 * 64] = rt_mark_draw(E, acc);
                waiting &= ~(1u << s1);
            }
        }
        const bool absorbed = d1 == __builtin_inf();
        // the next firing would come after a rate breakpoint (Eq. 28)
        const bool brk = SCHED && live && b_next < t_end && t_new > b_next;
        const bool term = !brk && (absorbed || t_new > t_end);
        const bool event = live && !term && !brk;
        // ---- the jump v_mu, checked against [0, 2^31 - 1] by lanes < |v_mu|
        const bool has_nu = event && li < nu_stride && nv.x >= 0;
        int64_t xv = 0;
        if (has_nu) xv = (int64_t)X[nv.x] + nv.y;
        const bool okl = xv >= 0 && xv <= 0x7FFFFFFF;
        // (in all these tests a frozen or unstarted group counts as rare)
        const unsigned long long bad = __ballot(!okl);
        const bool rare = !live || !(t_new <= t_end) || near || clamped || s_next < t_new || brk;
        if (__builtin_expect((__ballot(rare) | bad) != 0ull, 0)) {
            const bool ok = (bad & gmask) == 0ull;
            const bool near_tie = event && near;
            // Counted once per event: when another group of the wavefront
            // stops or meets a breakpoint, this group repeats its pass below
            // without applying its event, so the counters are bumped only once
            // the event is known to be applied (or, for a near-tie, when the
            // event ends the trajectory by an overflow, as the oracle counts
            // it); tie and the samples are idempotent.
            if (event) {
                if (near_tie) tie = tie == kTieNone ? fired : tie;
                while (s_next < t_new) {
                    if (it->samples) {
                        int32_t* dst = it->samples + r * it->ss_r + (int64_t)g * it->ss_g;
                        for (int j = li; j < N; j += L) dst[j * it->ss_n] = X[j];
                    }
                    ++g;
                    s_next = g < it->G ? rt_const(it->s)[g] : __builtin_inf();
                }
            }
            const bool stop = !live || term || !ok;
            if (near_tie && stop && li == 0) atomicAdd(&ws->near_ties, 1ull);   // event && !ok
            if (stop && !fresh) {
                // ---- end of the trajectory
                const int st = capped ? RTSSA_TRAJ_MAX_FIRINGS
                                      : (absorbed ? RTSSA_TRAJ_ABSORBED
                                                  : (term ? RTSSA_TRAJ_OK : RTSSA_TRAJ_OVERFLOW));
                const bool good = st == RTSSA_TRAJ_OK || st == RTSSA_TRAJ_ABSORBED;
                if (it->samples) {
                    for (; g < it->G; ++g) {
                        int32_t* dst = it->samples + r * it->ss_r + (int64_t)g * it->ss_g;
                        for (int j = li; j < N; j += L) dst[j * it->ss_n] = good ? X[j] : -1;
                    }
                }
                const double dt = t_end - t;
                unsigned long long left = 0ull;              // marked draws that no firing took
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int k = li + s * L;
                    if (k < M) {
                        if (good) T[s] = fma(la[s * 64], dt, T[s]);
                        if (it->n_out) it->n_out[r * M + k] = lnk[s * 64];
                        if (it->T_out) it->T_out[r * M + k] = T[s];
                        if (!((waiting >> s) & 1u) && le[s * 64] < 0.0) ++left;
                    }
                }
                if (left) atomicAdd(&ws->slow_logs, 0ull - left);
                if (it->x_final)
                    for (int j = li; j < N; j += L) it->x_final[r * N + j] = X[j];
                if (li == 0) {
                    if (it->t_last) it->t_last[r] = t;
                    if (it->status) it->status[r] = (uint8_t)st;
                    if (it->seq_hash) it->seq_hash[r] = hash;
                    if (it->tie_step) it->tie_step[r] = tie;
                    share.finished(fired, st);
                }
            }
            if (stop) {
                // ---- take the next trajectory unit
                unsigned long long u = 0;
                if (li == 0) u = (unsigned long long)share.take(&ws->next_unit, total);
                u = __shfl(u, gbase, 64);
                rt_wave_lds_fence();                          // X is reused
                fresh = false;
                capped = false;
                active = (int64_t)u < total;
                if (active) {
                    const int item = rt_find_item(unit_start, C.count, (int64_t)u);
                    it = rt_const(C.items) + item;
                    r = (int64_t)u - unit_start[item];
                    M = it->net.M;
                    N = it->net.N;
                    t_end = it->t_end;
                    net_id = it->net_id;
                    traj = it->traj_offset + (uint32_t)r;
                    const int32_t* x0 = it->x0 + (it->x0_per_traj ? r * N : 0);
                    for (int j = li; j < N; j += L) X[j] = x0[j];
                    t = 0.0;
                    g = 0;
                    s_next = it->G > 0 ? rt_const(it->s)[0] : __builtin_inf();
                    piece = 0;
                    b_next = SCHED && it->net.sched_B > 0 ? rt_const(it->net.sched_t)[0]
                                                          : __builtin_inf();
                    fired = 0;
                    tie = kTieNone;
                    hash = kFnvOffset;
                    waiting = 0u;
                    rt_wave_lds_fence();
                    // first internal firing times E(k, 0) and next draws E(k, 1)
                    // (the two words of one block) and propensities, one slot at
                    // a time; a slot past M keeps P = +inf, a = 0
                    bool plain = true;
#pragma unroll 1
                    for (int s1 = 0; s1 < S; ++s1) {
                        const int k = li + s1 * L;
                        double p0 = __builtin_inf(), an = 0.0;
                        if (k < M) {
                            const rt_u4 w =
                                rt_philox4x32_10(rt_u4{0u, (uint32_t)k, traj, net_id}, key0, key1);
                            p0 = rt_neglog_wave((((uint64_t)w.y << 32) | w.x) >> 11, false,
                                                &ws->slow_logs, sc);
                            bool acc;
                            const double e1 = rt_neglog_wave((((uint64_t)w.w << 32) | w.z) >> 11,
                                                             false, &ws->slow_logs, sc, &acc);
                            le[s1 * 64] = rt_mark_draw(e1, acc);
                            const double c = rt_const(it->net.c)[k];
                            an = rt_propensity_mem(rt_const(it->net.react)[k], c, X);
                            plain = plain && rt_plain_rate(c);
                        }
                        la[s1 * 64] = an;
                        linv[s1 * 64] = __builtin_amdgcn_rcpf((float)an);
                        lnk[s1 * 64] = 0u;
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            P[s] = s == s1 ? p0 : P[s];
                            T[s] = 0.0;
                        }
                    }
                    g_min = (__ballot(!plain) & gmask) ? __builtin_inff() : 1e-30f;
                    rt_wave_lds_fence();
                }
            }
            if (SCHED && brk) {
                // the clocks run to the breakpoint at the old rates, then
                // every propensity takes the new ones
                const double db = b_next - t;
                const rt_cptr<double> cr = rt_const(net->sched_c) + (size_t)piece * M;
                t = b_next;
                ++piece;
                b_next = piece < net->sched_B ? rt_const(net->sched_t)[piece]
                                              : __builtin_inf();
                bool plain = true;
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int k = li + s * L;
                    T[s] = fma(la[s * 64], db, T[s]);
                    if (k < M) {
                        const double an = rt_propensity_mem(rt_const(net->react)[k], cr[k], X);
                        la[s * 64] = an;
                        linv[s * 64] = __builtin_amdgcn_rcpf((float)an);
                        plain = plain && rt_plain_rate(cr[k]);
                    }
                }
                g_min = (__ballot(!plain) & gmask) ? __builtin_inff() : 1e-30f;
                rt_wave_lds_fence();
            }
            // started groups compute first gaps, groups past a breakpoint
            // solve again; the others repeat their (idempotent) pass
            if (__ballot(stop || brk) != 0ull) continue;
            // the event is applied below
            if (near_tie && li == 0) atomicAdd(&ws->near_ties, 1ull);
            if (clamped) atomicAdd(&ws->clamps, 1ull);
        }
        // ---- the event: internal clocks, the fired channel's next draw
#pragma unroll
        for (int s = 0; s < S; ++s) T[s] = fma(la[s * 64], d1, T[s]);
        if (own) {
            const double E = le[sm * 64];
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (sm == s) rt_land(T[s], P[s], E);
            lnk[sm * 64] += 1u;
            waiting |= 1u << sm;
        }
        // ---- new propensities of mu and D(mu) from the records: X before the
        // jump plus the record's changes
        auto touch = [&](const int4& e, double c, const int2& dl) {
            if (e.x >= 0) {
                const int kind = (int)((uint32_t)e.y >> 29);
                int32_t v0 = 0, v1 = 0;
                if (kind != RT_H_ZERO) v0 = X[e.y & RT_SPECIES_MASK] + dl.x;
                if (kind == RT_H_TWO) v1 = X[e.z] + dl.y;
                const double an = rt_propensity_counts(kind, (uint32_t)v0, (uint32_t)v1, c);
                const int o = at(e.x);
                la[o] = an;
                linv[o] = __builtin_amdgcn_rcpf((float)an);
            }
        };
        // (with a schedule the rates in force come from the piece)
        const rt_cptr<double> crate =
            SCHED && piece > 0 ? rt_const(net->sched_c) + (size_t)(piece - 1) * M
                               : rt_const(net->c);
#pragma unroll
        for (int q = 0; q < kR; ++q)
            touch(rec[q], SCHED ? crate[max(rec[q].x, 0)] : rc[q], rd[q]);
        if constexpr (kR * L < 64) {
            const int rows = min(n_other, 63) + 1;
            for (int q = kR * L; q < rows; q += L) {
                const int o = mr * 64 + q + li;              // (q + li < 64)
                const int4 e = rt_const(net->grow)[o];
                touch(e, SCHED ? crate[max(e.x, 0)] : rt_const(net->growc)[o],
                      rt_const(net->gdel)[o]);
            }
        }
        if (has_nu) X[nv.x] = (int32_t)xv;
        rt_wave_lds_fence();
        if (__builtin_expect(n_other > 63, 0)) {
            // more than 63 others: the rest of the CSR list D(mu) (rare)
            const int de = rt_const(net->dep_ptr)[mu + 1];
            for (int q = rt_const(net->touch_more)[mu] + li; q < de; q += L) {
                const int k = rt_const(net->dep_idx)[q];
                const double an = rt_propensity_mem(rt_const(net->react)[k], crate[k], X);
                const int o = at(k);
                la[o] = an;
                linv[o] = __builtin_amdgcn_rcpf((float)an);
            }
            rt_wave_lds_fence();
        }
        t = t_new;
        ++fired;
        hash = (hash ^ (unsigned long long)(uint32_t)mu) * kFnvPrime;
        capped = fired >= C.max_firings;
    }
    share.flush(ws);
}

typedef void (*subwave_kernel_t)(rt_class_dev);

template <int L, int S>
subwave_kernel_t sw_pick(bool sched)
{
    return sched ? rt_subwave_kernel<L, S, true> : rt_subwave_kernel<L, S, false>;
}

subwave_kernel_t select_subwave(int L, int S, bool sched)
{
#define RT_CASE(l, s) if (L == l && S == s) return sw_pick<l, s>(sched);
    RT_CASE(4, 2) RT_CASE(4, 4) RT_CASE(4, 5) RT_CASE(4, 6) RT_CASE(4, 8)
    RT_CASE(8, 2) RT_CASE(8, 4) RT_CASE(8, 5) RT_CASE(8, 6) RT_CASE(8, 8)
    RT_CASE(16, 2) RT_CASE(16, 4) RT_CASE(16, 5) RT_CASE(16, 6) RT_CASE(16, 8)
    RT_CASE(32, 2) RT_CASE(32, 4) RT_CASE(32, 5) RT_CASE(32, 6) RT_CASE(32, 8)
    RT_CASE(64, 2) RT_CASE(64, 4) RT_CASE(64, 5) RT_CASE(64, 6) RT_CASE(64, 8)
#undef RT_CASE
    return nullptr;
}

}  // namespace

// Lanes per trajectory for an M-channel network: the fewest lanes that keep
// at most 8 channels per lane (at least 4 lanes).
int rt_subwave_lanes(int M)
{
    int L = 4;
    while (L < 64 && L * 8 < M) L <<= 1;
    return L;
}

// Slots per lane: the fewest of 2, 4, 5, 6, 8 that hold M channels (0: none).
int rt_subwave_slots(int M, int L)
{
    const int s = (M + L - 1) / L;
    return s <= 2 ? 2 : (s <= 4 ? 4 : (s <= 6 ? s : (s <= 8 ? 8 : 0)));
}

// LDS bytes of a workgroup of `waves` wavefronts: the dynamic part the launch asks
// for, and with the logarithm table and the wavefronts' shares.
static size_t dynamic_lds_bytes(int waves, int L, int S, int N)
{
    return waves * wave_lds_bytes(L, S, (N + 3) & ~3);
}

static size_t group_lds_bytes(int waves, int L, int S, int N)
{
    constexpr size_t fixed = sizeof(rt_log_lds<kWaves>) + kWaves * sizeof(rt_wave_share);
    return (fixed + 15) / 16 * 16 + dynamic_lds_bytes(waves, L, S, N);
}

// A workgroup's LDS limit, which is also a CU's LDS (0: no device answers).
static size_t lds_limit()
{
    int dev = 0, bytes = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return 0;
    return (size_t)bytes;
}

// Wavefronts per workgroup: the number that leaves a CU's LDS the most wavefronts
// (0: not one fits), the larger of equals; *cu: that most.  2 at 8 slots and 4
// below while the counts X are small beside the channels' state; fixed at those,
// networks of many species lost to idle SIMDs (16000 trajectories: 250 channels,
// 1500 species 17.1 ms, 11.5 this way; 400, 3000 31.0 and 20.7; 128, 800 8.3 and
// 5.5).
static int group_waves(size_t limit, int L, int S, int N, int* cu)
{
    int best = 0;
    *cu = 0;
    for (int w = kWaves; w >= 1; --w) {
        const int n = std::min(w * (int)(limit / group_lds_bytes(w, L, S, N)),
                               4 * subwave_min_waves(S));
        if (n > *cu) {
            *cu = n;
            best = w;
        }
    }
    return best;
}

// Whether L lanes a trajectory leave every SIMD of a CU a wavefront beside N
// species, for any network of M's slot range (a batch's class runs its networks
// with the most slots of one and the most species of another).  More lanes are
// more wavefronts of fewer trajectories, about as many trajectories in all.
bool rt_subwave_fits(int M, int N, int L)
{
    int cu = 0;
    const size_t limit = lds_limit();
    if (limit) group_waves(limit, L, rt_subwave_slots(M, L) <= 4 ? 4 : 8, N, &cu);
    return limit == 0 || cu >= 4;
}

// Lanes per trajectory when nothing else says: as many as keep the units'
// wavefronts within waves_per_cu, at least 8 and rt_subwave_lanes, and as many
// as the species call for (so whether a network runs does not depend on the
// units).  More lanes are fewer slots and fewer groups a wavefront, so a faster
// firing, while a wavefront has its SIMD to itself; on a full device fewer lanes
// do more per instruction (45 channels, lanes 8 / 16 / 32 / 64: 300 trajectories 3.7 / 2.8
// / 2.6 / 2.4 ms, 3000 3.8 / 2.9 / 3.4 / 3.7 ms, 30000 7.2 / 8.9 / 13.4 / 22.6
// ms; 20 channels at 4 lanes: 2.6, 2.7 and 3.3 ms against 1.7, 1.7 and 2.7 at 8).
int rt_subwave_auto_lanes(int M, int N, int64_t units, int waves_per_cu)
{
    int L = std::max(8, rt_subwave_lanes(M));
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return L;
    while (L < 64 && units * (2 * L) <= (int64_t)cus * waves_per_cu * 64) L <<= 1;
    while (L < 64 && !rt_subwave_fits(M, N, L)) L <<= 1;
    return L;
}

int rt_launch_subwave(int max_M, const rt_class_dev& C, int L, int grid, hipStream_t stream,
                      int* grid_used)
{
    const int S = rt_subwave_slots(max_M, L);
    subwave_kernel_t kfn = select_subwave(L, S, C.has_schedule != 0);
    if (!kfn) return rt_fail(RTSSA_E_UNSUPPORTED, "no sub-wave kernel for this size");
    const size_t limit = lds_limit();
    if (limit == 0) return rt_fail(RTSSA_E_HIP, "device query failed");
    int cu_waves = 0;
    const int waves = group_waves(limit, L, S, C.max_N, &cu_waves);
    if (waves == 0) return rt_fail(RTSSA_E_UNSUPPORTED, "sub-wave LDS too large");
    const int block = 64 * waves;
    const size_t lds = dynamic_lds_bytes(waves, L, S, C.max_N);
    if (lds > 48 * 1024 &&
        hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds) != hipSuccess)
        return rt_fail(RTSSA_E_HIP, "cannot raise the LDS limit");
    if (grid <= 0) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return rt_fail(RTSSA_E_HIP, "device query failed");
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, block, lds) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        grid = cus * per_cu;
    }
    if (grid_used) *grid_used = grid;
    hipLaunchKernelGGL(kfn, dim3(grid), dim3(block), lds, stream, C);
    return hipGetLastError() == hipSuccess ? RTSSA_OK
                                           : rt_fail(RTSSA_E_HIP, "sub-wave kernel launch failed");
}
