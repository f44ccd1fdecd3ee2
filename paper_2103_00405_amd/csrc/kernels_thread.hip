// kernels_thread.hip -- thread-per-trajectory mapping for small networks.
//
// One lane owns one trajectory at a time; its whole state (t, X, and per
// channel T_k, P_k, a_k, 1/a_k, n_k) lives in VGPRs, the network constants of
// the wavefront's current item in SGPRs.  The grid is persistent: a lane that
// finishes a trajectory takes the next trajectory of the same item from a
// device counter, so lanes stay busy despite uneven trajectory lengths; a
// wavefront moves to another item only when all of its lanes are idle.
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

// fn(x[j]) for a wave-uniform j (a species index of the network): a switch
// becomes scalar branches, so x stays in registers instead of being copied
// to scratch memory for an indexed load, and each branch works on its own
// register rather than on a copy of it.
template <int NT, class F>
__device__ __forceinline__ void with_species(const double (&x)[NT], int j, F fn)
{
    switch (j) {
        case 1: if constexpr (NT > 1) { fn(x[1]); return; } break;
        case 2: if constexpr (NT > 2) { fn(x[2]); return; } break;
        case 3: if constexpr (NT > 3) { fn(x[3]); return; } break;
        case 4: if constexpr (NT > 4) { fn(x[4]); return; } break;
        case 5: if constexpr (NT > 5) { fn(x[5]); return; } break;
        case 6: if constexpr (NT > 6) { fn(x[6]); return; } break;
        case 7: if constexpr (NT > 7) { fn(x[7]); return; } break;
        default: break;
    }
    fn(x[0]);
}

// The rate constant as propensities() uses it: halved for a homodimer
// (exact: c is 0 or at least 1e-280).
__device__ __forceinline__ double kernel_rate(int kind, double c)
{
    return kind == RT_H_PAIR ? 0.5 * c : c;
}

// a_k = RN(c_k RN(h_k)) of Eq. 1-2 for every channel, the kinds wave-uniform
// and X in registers.  Counts are below 2^31, so a product of two is exact
// before its one rounding: RN(X_i X_j) is the binary64 product, and a
// homodimer's 2 RN(h) = RN(X^2 - X) one fma (+0 for X = 0 and 1), its factor
// 1/2 in the rate; no 64-bit integer product and one conversion per species.
template <int MT, int NT>
__device__ __forceinline__ void propensities(const int (&kind)[MT], const int (&s0)[MT],
                                             const int (&s1)[MT], const double (&c)[MT],
                                             const int32_t (&X)[NT], double (&a)[MT])
{
    double x[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) x[j] = (double)(uint32_t)X[j];
#pragma unroll
    for (int k = 0; k < MT; ++k) {
        if (kind[k] == RT_H_ZERO) {
            a[k] = c[k];
        } else if (kind[k] == RT_H_ONE) {
            with_species<NT>(x, s0[k], [&](double u) { a[k] = c[k] * u; });
        } else if (kind[k] == RT_H_PAIR) {
            with_species<NT>(x, s0[k], [&](double u) { a[k] = c[k] * fma(u, u, -u); });
        } else if constexpr (NT == 2) {
            a[k] = c[k] * (x[0] * x[1]);
        } else {
            double u = 0.0;
            with_species<NT>(x, s0[k], [&](double v) { u = v; });
            with_species<NT>(x, s1[k], [&](double v) { a[k] = c[k] * (u * v); });
        }
    }
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

// Collects one lane's writes to one 64-byte line in its LDS buffer and
// stores them together when the next write falls in another line (or on
// flush); only the words the lane wrote are stored.
struct rt_line_writer {
    int32_t* buf;       // 16 words of LDS
    uint64_t line;      // address >> 6 of the buffered line (~0: none)
    uint32_t mask;      // words written

    __device__ __forceinline__ void flush()
    {
        if (mask) {
            int32_t* const base = (int32_t*)(line << 6);
#pragma unroll
            for (int w = 0; w < 16; ++w)
                if (mask & (1u << w)) base[w] = buf[w];
            mask = 0u;
        }
    }

    __device__ __forceinline__ void put(int32_t* p, int32_t v)
    {
        const uint64_t addr = (uint64_t)p;
        if ((addr >> 6) != line) {
            flush();
            line = addr >> 6;
        }
        const int w = (int)((addr >> 2) & 15u);
        buf[w] = v;
        mask |= 1u << w;
    }
};

// One wavefront's share of the trajectory counter and of the run's counts, in
// LDS.  Lanes take trajectories from the reserved range [next, end); when a
// pass needs more than are left, one lane reserves as many as the stopping
// lanes need, and more while many trajectories are left (a quarter of an even
// share of the rest, at most 64).  Firings and end states are summed here and
// added to the run's counters once, when the wavefront ends.  With one
// device-wide atomic per trajectory for the trajectory and two for the counts,
// all on one line, ensembles of short trajectories were bound by those: the
// expectation and gradient of a birth-death process over 2^18 trajectories of
// 200 firings took 5.73 ms, 2.25 ms this way.
struct rt_wave_share {
    int64_t next, end;
    unsigned long long firings;
    uint32_t status[4];

    // A wavefront that runs its item alone (a batch) owns every trajectory.
    __device__ __forceinline__ void start_item(bool own)
    {
        if ((threadIdx.x & 63u) == 0) {
            next = 0;
            end = own ? INT64_MAX : 0;
        }
        rt_wave_lds_fence();
    }

    // The next trajectory of each active lane (>= R: none left).
    __device__ __forceinline__ int64_t take(unsigned long long* ctr, int64_t R)
    {
        const unsigned long long takers = __ballot(true);
        const int want = __popcll(takers);
        const int rank = __popcll(takers & ((1ull << (threadIdx.x & 63u)) - 1ull));
        const int64_t n0 = next, e0 = end, left = e0 - n0;
        int64_t r = n0 + rank;
        rt_wave_lds_fence();
        if (left < want) {                                 // the same in every lane
            const float waves = (float)(gridDim.x * (blockDim.x >> 6));
            const int share = (int)fminf((float)(R - e0) * 0.25f / waves, 64.0f);
            const int n = max(want - (int)left, share);
            unsigned long long at = 0;
            if (rank == 0) at = atomicAdd(ctr, (unsigned long long)n);
            at = rt_first_lane_u64(at);
            if (rank >= left) r = (int64_t)at + (rank - left);
            if (rank == 0) {
                next = (int64_t)at + (want - left);
                end = (int64_t)at + n;
            }
        } else if (rank == 0) {
            next = n0 + want;
        }
        rt_wave_lds_fence();
        return r;
    }

    __device__ __forceinline__ void clear()
    {
        if ((threadIdx.x & 63u) == 0) {
            firings = 0ull;
            for (int q = 0; q < 4; ++q) status[q] = 0u;
        }
        rt_wave_lds_fence();
    }

    __device__ __forceinline__ void finished(uint32_t fired, int st)
    {
        atomicAdd(&firings, (unsigned long long)fired);
        atomicAdd(&status[st], 1u);
    }

    __device__ __forceinline__ void flush(rt_ws* ws)
    {
        rt_wave_lds_fence();
        if ((threadIdx.x & 63u) == 0) {
            if (firings) atomicAdd(&ws->firings, firings);
            for (int q = 0; q < 4; ++q)
                if (status[q]) atomicAdd(&ws->status_count[q], (unsigned long long)status[q]);
        }
    }
};

// Waves per SIMD each instantiation is compiled for: the most at which its
// state (X, n, a and, for the random-time method, T, P and 1/a, in registers;
// the network in SGPRs; with a rate schedule, the lane's rates too) fits
// without spilling to scratch.
constexpr int thread_min_waves(int MT, int NT, int METHOD, bool SCHED)
{
    if (METHOD == RTSSA_METHOD_DIRECT) return 4;
    // 5 waves fit without scratch up to 3 channels and 2 species (and 2 x 4);
    // on the Lotka-Volterra ensemble they measured 2.7 % faster than 4
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
    // per-lane buffer of one 64-byte line of sample output: a lane's sample
    // row is written a few bytes at a time, at its own event times; collecting
    // the words of a line and storing them together lets the L2 write each
    // line back once instead of once per sample point
    __shared__ int32_t line_buf[256][16];
    int32_t* const lb = line_buf[threadIdx.x];
    __shared__ rt_wave_share wave_shares[4];
    rt_wave_share& share = wave_shares[threadIdx.x >> 6];
    share.clear();
    // firing counts n_k of the lane's trajectory: the count behind the next draw
    // comes from one LDS atomic instead of selects over every channel's register
    __shared__ uint32_t counts[MT][256];
    uint32_t* const cnt = &counts[0][threadIdx.x];

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
        int kind[MT], s0[MT], s1[MT], nu[MT][NT];
        double c[MT];
#pragma unroll
        for (int k = 0; k < MT; ++k) {
            if (k < net.M) {
                int2 rr = rt_const(net.react)[k];
                kind[k] = (int)((uint32_t)rr.x >> 29);
                s0[k] = rr.x & RT_SPECIES_MASK;
                s1[k] = rr.y;
                c[k] = kernel_rate(kind[k], rt_const(net.c)[k]);
            } else {
                kind[k] = RT_H_ZERO; s0[k] = 0; s1[k] = 0; c[k] = 0.0;   // dead padding channel
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
        // counts up to here are safe from any jump's increase
        int32_t up = 0;
#pragma unroll
        for (int k = 0; k < MT; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) up = max(up, nu[k][j]);
        const uint32_t x_safe = 0x7FFFFFFFu - (uint32_t)up;

        // ---- trajectory state
        int32_t X[NT];
        double T[MT], Pk[MT], a[MT];
        rt_traj_words tw{0u, 0u};
#pragma unroll
        for (int j = 0; j < NT; ++j) X[j] = 0;
#pragma unroll
        for (int k = 0; k < MT; ++k) { T[k] = 0.0; Pk[k] = 0.0; a[k] = 0.0; }
        double t = 0.0, s_next = 0.0;
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
        uint32_t fired = 0, tie = kTieNone, traj = 0;
        unsigned long long hash = kFnvOffset;
        int64_t r = 0;

        rt_line_writer lw{lb, ~0ull, 0u};
        auto write_sample = [&](int32_t gg, bool invalid) {
            int32_t* dst = it->samples + r * it->ss_r + (int64_t)gg * it->ss_g;
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (j < N) lw.put(dst + j * it->ss_n, invalid ? -1 : X[j]);
        };
        auto refresh = [&]() {
            if constexpr (SCHED) propensities<MT, NT>(kind, s0, s1, cl, X, a);
            else propensities<MT, NT>(kind, s0, s1, c, X, a);
        };

        // Each pass is one firing of every active lane, bound by VALU issue on a
        // full device (92 % busy): 209 instructions a firing on the Lotka-Volterra
        // ensemble, 947 ms for 2^20 trajectories, where three exact gaps, selects
        // for every update and integer products took 307 and (with the same
        // logarithm) 1059 ms.  The common path is
        // straight-line; every rare event (start or end of a trajectory, a
        // sample point, a near-tie, a clamped gap, an overflow, the firing
        // cap) is handled in one branch entered only when some lane of the
        // wave needs it.
        bool active = true, fresh = true, capped = false;
        while (active) {
            bool f[MT];                                    // the channel that fires
            double d1 = 0.0;
            bool near = false, clamped = false;
            int mu = 0;
            if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                // The argmin of the gaps (Eq. 25).  Only the smallest gap's value
                // enters the trajectory, so the gaps are first compared in
                // binary32, (P - T) rcp(a) with relative error below 2^-21, and
                // the one exact reciprocal RN(1 / a_mu) is made for the winner:
                // three IEEE divisions per firing (63 issue cycles each) were 15 %
                // of the Lotka-Volterra kernel's issue time.
                // The binary32 order decides when the smallest is positive and
                // the second at least 1 + 2^-18 times it plus 1e-30 (which also
                // excludes near-ties, clamped gaps and values whose binary32
                // form under- or overflowed); else, and for the rare event that
                // needs d2, the exact form below decides.
                double df[MT];
                float gf[MT];
#pragma unroll
                for (int k = 0; k < MT; ++k) {
                    df[k] = Pk[k] - T[k];
                    gf[k] = (float)df[k] * __builtin_amdgcn_rcpf((float)a[k]);
                }
                float g1, g2;
                rt_two_smallest<MT>(gf, g1, g2);
                const bool amb = !(g1 > 0.0f) || !(g2 > fmaf(g1, 1.0f + 0x1p-18f, 1e-30f));
                if (__builtin_expect(__ballot(amb) != 0ull, 0)) {
                    if (amb) {
                        // exact gaps: max(0, RN((P - T) RN(1 / a))), +inf for a
                        // frozen channel, lowest k on ties
                        rt_min2 sel{__builtin_inf(), __builtin_inf(), 0};
#pragma unroll
                        for (int k = 0; k < MT; ++k) {
                            const double raw = df[k] * (1.0 / a[k]);
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
                            clamped = clamped || (neg && df[k] * (1.0 / a[k]) < 0.0);
                            df[k] = neg ? 0.0 : df[k];
                        }
                    }
                }
                double am = a[MT - 1], dm = df[MT - 1];
                mu = MT - 1;
                f[MT - 1] = true;
#pragma unroll
                for (int k = MT - 2; k >= 0; --k) {
                    f[k] = gf[k] == g1;
                    am = f[k] ? a[k] : am;
                    dm = f[k] ? df[k] : dm;
                    mu = f[k] ? k : mu;
                    f[MT - 1] = f[MT - 1] && !f[k];
                }
                d1 = dm * rt_recip(am);
            } else {
                // direct method: total rate, one block for the waiting time and
                // the search (padding channels add +0 and are never reached)
                double a0 = 0.0;
#pragma unroll
                for (int k = 0; k < MT; ++k) a0 += a[k];
                const rt_u4 w = rt_philox4x32_10(rt_u4{fired, 0xFFFFFFFFu, traj, net_id}, key0, key1);
                const uint64_t m1 = (((uint64_t)w.y << 32) | w.x) >> 11;
                const uint64_t m2 = (((uint64_t)w.w << 32) | w.z) >> 11;
                const double E1 = rt_neglog_wave(m1, false, &ws->slow_logs, sc);
                d1 = a0 == 0.0 ? __builtin_inf() : E1 / a0;
                const double target = (double)(m2 + 1) * 0x1p-53 * a0;
                double run = 0.0;
                bool found = false;
                mu = MT - 1;
#pragma unroll
                for (int k = 0; k < MT; ++k) {
                    run += a[k];
                    f[k] = !found && (run >= target || k == MT - 1);
                    mu = f[k] ? k : mu;
                    found = found || f[k];
                }
            }
            const double t_new = t + d1;
            // a jump may leave [0, 2^31 - 1] only upwards (a channel with a_k > 0
            // has its reactants), and only from a count past x_safe
            uint32_t x_top = (uint32_t)X[0];
#pragma unroll
            for (int j = 1; j < NT; ++j) x_top = max(x_top, (uint32_t)X[j]);
            // (NaN, from an absorbed state, is past every time)
            if (__builtin_expect((__ballot(!(t_new <= t_stop)) | __ballot(x_top > x_safe) |
                                  __ballot(near) | __ballot(clamped)) != 0ull, 0)) {
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
                    for (int k = 0; k < MT - 1; ++k) dl = f[k] ? nu[k][j] : dl;
                    sign |= (int32_t)((uint32_t)X[j] + (uint32_t)dl);
                }
                const bool ok = sign >= 0;
                const bool event = live && !term && !brk;     // this pass may apply an event
                // Counted once per event: when another lane of the wave stops or
                // meets a breakpoint, this lane repeats its pass below without
                // applying its event, so the counters are bumped only once the
                // event is known to be applied (or, for a near-tie, when the
                // event ends the trajectory by an overflow, as the oracle counts
                // it); tie and the samples are idempotent.
                const bool near_tie = event && near;
                if (event) {
                    if (near_tie) tie = tie == kTieNone ? fired : tie;
                    while (s_next < t_new) {
                        if (it->samples) write_sample(g, false);
                        ++g;
                        s_next = g < it->G ? it->s[g] : __builtin_inf();
                    }
                    t_stop = fmin(s_next, SCHED ? fmin(b_next, t_end) : t_end);
                }
                if (SCHED && brk) {
                    // every internal clock runs to the breakpoint at the old
                    // rates; the propensities take the next piece's rates
                    const double db = b_next - t;
#pragma unroll
                    for (int k = 0; k < MT; ++k) T[k] = fma(a[k], db, T[k]);
                    t = b_next;
#pragma unroll
                    for (int k = 0; k < MT; ++k)
                        cl[k] = k < M ? kernel_rate(kind[k], sched_c[piece * M + k]) : 0.0;
                    ++piece;
                    b_next = piece < sB ? sched_t[piece] : __builtin_inf();
                    t_stop = fmin(s_next, fmin(b_next, t_end));
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
                    if (it->samples) {
                        for (int32_t gg = g; gg < it->G; ++gg) write_sample(gg, !good);
                        lw.flush();
                    }
                    if (METHOD == RTSSA_METHOD_RANDOM_TIME && good) {
                        const double dt = t_end - t;
#pragma unroll
                        for (int k = 0; k < MT; ++k) T[k] = fma(a[k], dt, T[k]);
                    }
                    if (it->n_out) {
#pragma unroll
                        for (int k = 0; k < MT; ++k) if (k < M) it->n_out[r * M + k] = cnt[k * 256];
                    }
                    if (METHOD == RTSSA_METHOD_RANDOM_TIME && it->T_out) {
#pragma unroll
                        for (int k = 0; k < MT; ++k) if (k < M) it->T_out[r * M + k] = T[k];
                    }
                    if (it->x_final) {
#pragma unroll
                        for (int j = 0; j < NT; ++j) if (j < N) it->x_final[r * N + j] = X[j];
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
                        r = rr;
                        traj = traj_offset + (uint32_t)rr;
                        const int32_t* x0 = it->x0 + (it->x0_per_traj ? rr * N : 0);
#pragma unroll
                        for (int j = 0; j < NT; ++j) X[j] = j < N ? x0[j] : 0;
                        t = 0.0;
                        g = 0;
                        s_next = it->G > 0 ? it->s[0] : __builtin_inf();
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
#pragma unroll
                            for (int k = 0; k < MT; ++k) T[k] = 0.0;
                            // first internal firing times, one draw at a time
#pragma unroll 1
                            for (int k = 0; k < MT; ++k) {
                                const double E0 = rt_exp1_wave(key0, key1, traj, net_id,
                                                               (uint32_t)k, 0u, &ws->slow_logs, sc);
#pragma unroll
                                for (int q = 0; q < MT; ++q) Pk[q] = q == k ? E0 : Pk[q];
                            }
                        }
                    }
                }
                // started lanes (and lanes past a breakpoint) compute their gaps
                if (__ballot(stop || brk) != 0ull) continue;
                // the event is applied below
                if (near_tie) atomicAdd(&ws->near_ties, 1ull);
                if (clamped) atomicAdd(&ws->clamps, 1ull);
            }
            t = t_new;
            ++fired;
            if (want_hash) hash = (hash ^ (unsigned long long)(uint32_t)mu) * kFnvPrime;
            // the fired channel's updates run under its lanes' mask, one
            // instruction each (as selects over the channels the internal times
            // and the jump took six a channel and two a species); the empty
            // statements keep them from becoming selects again
            if constexpr (METHOD == RTSSA_METHOD_RANDOM_TIME) {
                // internal times advance by a_k Delta (Eq. 15); the fired channel
                // lands exactly on its firing internal time and draws the next
                const uint32_t n_mu = atomicAdd(&cnt[mu * 256], 1u) + 1u;
#pragma unroll
                for (int k = 0; k < MT; ++k) T[k] = fma(a[k], d1, T[k]);
                const uint64_t m = rt_block_m53(
                    rt_philox_traj(tw, n_mu >> 1, (uint32_t)mu, net_k1, key0, key1), n_mu);
                const double E = rt_neglog_wave(m, false, &ws->slow_logs, sc);
#pragma unroll
                for (int k = 0; k < MT; ++k)
                    if (f[k]) {
                        asm volatile("");
                        T[k] = Pk[k];
                        Pk[k] = Pk[k] + E;
#pragma unroll
                        for (int j = 0; j < NT; ++j) X[j] += nu[k][j];
                    }
            } else {
                atomicAdd(&cnt[mu * 256], 1u);
#pragma unroll
                for (int k = 0; k < MT; ++k)
                    if (f[k]) {
                        asm volatile("");
#pragma unroll
                        for (int j = 0; j < NT; ++j) X[j] += nu[k][j];
                    }
            }
            refresh();
            if (__builtin_expect(__ballot(fired >= C.max_firings) != 0ull, 0)) {
                capped = fired >= C.max_firings;
                t_stop = capped ? -1.0 : t_stop;
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
int launch_mn(const rt_class_dev& C, int block, int grid, hipStream_t stream, int* grid_used,
              int64_t lanes_wanted, int method, bool sched)
{
    thread_kernel_t kfn = method == RTSSA_METHOD_DIRECT
                              ? rt_thread_kernel<MT, NT, RTSSA_METHOD_DIRECT, false>
                              : (sched ? rt_thread_kernel<MT, NT, RTSSA_METHOD_RANDOM_TIME, true>
                                       : rt_thread_kernel<MT, NT, RTSSA_METHOD_RANDOM_TIME, false>);
    if (grid <= 0) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return rt_fail(RTSSA_E_HIP, "device query failed");
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, block, 0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        int64_t need = (lanes_wanted + block - 1) / block;
        int64_t full = (int64_t)cus * per_cu;
        grid = (int)std::max<int64_t>(1, std::min<int64_t>(need, full));
    }
    if (grid_used) *grid_used = grid;
    hipLaunchKernelGGL(kfn, dim3(grid), dim3(block), 0, stream, C);
    return hipGetLastError() == hipSuccess ? RTSSA_OK : rt_fail(RTSSA_E_HIP, "thread kernel launch failed");
}

template <int MT>
int launch_m(int N, const rt_class_dev& C, int block, int grid, hipStream_t stream, int* gu,
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
// and absent species); lanes = trajectories wanted in flight.
int rt_launch_thread(int M, int N, const rt_class_dev& C, int block, int grid,
                     hipStream_t stream, int* grid_used, int64_t lanes, int method)
{
    const bool sched = C.has_schedule != 0;
    if (sched && method != RTSSA_METHOD_RANDOM_TIME)
        return rt_fail(RTSSA_E_UNSUPPORTED, "rate schedules run with the random-time method");
    if (!rt_thread_supported(M, N))
        return rt_fail(RTSSA_E_UNSUPPORTED, "network too large for the thread mapping");
    if (block <= 0) block = 256;
    if (block > 256 || block % 64)
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
