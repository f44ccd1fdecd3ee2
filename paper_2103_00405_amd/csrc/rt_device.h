// rt_device.h -- device-side wrappers of the numeric core for the kernels.
#pragma once
#define RT_HD __device__ __forceinline__
#define RT_LOG_CONST __constant__
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"
#include "rt_math.h"

constexpr uint32_t kTieNone = 0xFFFFFFFFu;                 // tie_step of a path without near-ties
constexpr unsigned long long kFnvOffset = 0xcbf29ce484222325ull;   // seq_hash start
constexpr unsigned long long kFnvPrime = 0x100000001b3ull;         // seq_hash multiplier

// Read-only launch data (network tables, item descriptors, prefix sums, the
// sample grid) read through the constant address space: the compiler may
// then treat the loads as invariant and, where the address is uniform, issue
// them as scalar loads into SGPRs.  Only for memory that no kernel of the
// launch writes.  (The host pass of this single-source file only parses the
// kernels; it sees plain pointers.)
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using rt_cptr = const __attribute__((address_space(4))) T*;
#else
template <typename T>
using rt_cptr = const T*;
#endif

template <typename T>
__device__ __forceinline__ rt_cptr<T> rt_const(const T* p)
{
    return (rt_cptr<T>)p;
}

// ---------------------------------------------------------------------
// Arithmetic of one channel and of the selection, shared by every kernel.

// RN((double)h) for h < 2^64: both halves convert exactly, one rounding.
__device__ __forceinline__ double rt_u64_to_f64(uint64_t h)
{
    return fma((double)(uint32_t)(h >> 32), 0x1p32, (double)(uint32_t)h);
}

// a_k = RN(c_k RN(h_k(X))) of Eq. 1-2 with h_k = prod_j C(X_j, sigma_jk)
// exact in 64-bit integers (C(X, 2) = X(X - 1) / 2); kind, s0 and s1 come
// from the reactant table (RT_H_*), x(j) reads species j.  One-species h is
// below 2^32 and converts exactly without the two-part form.
template <class XGet>
__device__ __forceinline__ double rt_propensity(int kind, int s0, int s1, double c, XGet x)
{
    uint64_t h;
    if (kind == RT_H_ZERO) {
        h = 1;
    } else if (kind == RT_H_ONE) {
        return c * (double)(uint32_t)x(s0);
    } else if (kind == RT_H_PAIR) {
        const uint32_t v = (uint32_t)x(s0);
        h = ((uint64_t)v * (uint32_t)(v - 1u)) >> 1;   // v = 0 gives 0
    } else {
        h = (uint64_t)(uint32_t)x(s0) * (uint32_t)x(s1);
    }
    return c * rt_u64_to_f64(h);
}

// The same from the reactant counts v0 = X_s0 and v1 = X_s1 (read only as
// the kind needs them), as selects rather than branches: lanes of one
// wavefront holding channels of different kinds take one path.  One-species h
// converts exactly either way, so the value is the one above.
__device__ __forceinline__ double rt_propensity_counts(int kind, uint32_t v0, uint32_t v1, double c)
{
    const uint64_t pair = ((uint64_t)v0 * (uint32_t)(v0 - 1u)) >> 1;
    const uint64_t two = (uint64_t)v0 * v1;
    const uint64_t h = kind == RT_H_ZERO ? 1ull
                     : kind == RT_H_ONE ? (uint64_t)v0
                     : kind == RT_H_PAIR ? pair : two;
    return c * rt_u64_to_f64(h);
}

// The same with X in memory (LDS) and the packed reactant-table entry
// rr = (s0 | kind << 29, s1), in the select form.
__device__ __forceinline__ double rt_propensity_mem(int2 rr, double c, const int32_t* X)
{
    const int kind = (int)((uint32_t)rr.x >> 29);
    int32_t v0 = 0, v1 = 0;
    if (kind != RT_H_ZERO) v0 = X[rr.x & RT_SPECIES_MASK];
    if (kind == RT_H_TWO) v1 = X[rr.y];
    return rt_propensity_counts(kind, (uint32_t)v0, (uint32_t)v1, c);
}

// RN(1 / a) for a normal a whose reciprocal is normal: v_rcp_f64 (2^-24.3),
// one cubic step to within an ulp, and the residual, exact in one fma, folded
// in with one rounding (Markstein's construction).  Seven instructions where
// the general division takes eleven.
__device__ __forceinline__ double rt_recip(double a)
{
    double y = __builtin_amdgcn_rcp(a);
    const double e = fma(-a, y, 1.0);
    y = fma(y, fma(e, e, e), y);
    return fma(fma(-a, y, 1.0), y, y);
}

// Rates for which every a_k > 0 is a normal binary32 number or overflows, and
// every gap too (h < 2^62, and 1e-32 < P - T < 37): 0 or 2^-100 .. 2^60.  The
// kernels that order gaps in binary32 take the exact form at every firing when
// some rate is outside.  That costs the thread and sub-wave kernels what their
// binary32 form saves (7 channels 8.4 ms for 3.7, 301 channels 5.8 for 3.3); the
// workgroup kernel, with its second barrier, would lose far more (2000 channels
// 9.3 ms for 3.4, 4.1 with binary64 gaps alone) and scales the rates first.
__device__ __forceinline__ bool rt_plain_rate(double c)
{
    return c == 0.0 || (c >= 0x1p-100 && c <= 0x1p60);
}

// A firing channel's internal times: T = P, then P += |E| (a draw waiting for
// its firing carries a mark in its sign, rt_mark_draw).  In place (the compiler
// adds into a temporary and copies) and never as selects.
__device__ __forceinline__ void rt_land(double& T, double& P, double E)
{
    asm volatile("v_mov_b64 %0, %1" : "=v"(T) : "v"(P));
    asm volatile("v_add_f64 %0, %0, |%1|" : "+v"(P) : "v"(E));
}

// A draw made ahead of its firing (sub-wave and workgroup kernels): negative when
// it took the accurate phase.  Such a draw is counted when it is made and, should
// the trajectory end without taking it, taken off again at the end (which draws
// are ever made ahead depends on the wavefront's other trajectories; which are
// taken does not).  The kernel adds |E| when the channel fires, a modifier of the
// addition.
__device__ __forceinline__ double rt_mark_draw(double E, bool accurate)
{
    return accurate ? -E : E;
}

// The near-tie rule (Eq. 4 gives ties probability zero; in binary64 the two
// smallest gaps d1 <= d2 can still round within reach of each other):
// RN(d2 - d1) <= RN(1e-12 d1).
__device__ __forceinline__ bool rt_near_tie(double d1, double d2)
{
    return d2 - d1 <= 1e-12 * d1;
}

// Orders the wavefront's LDS accesses (the hardware completes them in order
// for one wavefront; this keeps the compiler from reordering them).
__device__ __forceinline__ void rt_wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Index of the item owning global unit u: unit_start[i] <= u < unit_start[i+1].
__device__ __forceinline__ int rt_find_item(rt_cptr<int64_t> unit_start, int count, int64_t u)
{
    int lo = 0, hi = count;   // unit_start[lo] <= u < unit_start[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (unit_start[mid] <= u) lo = mid; else hi = mid;
    }
    return lo;
}

// A 64-bit value of the wavefront's first active lane, known to the compiler
// as the same in every lane (so that what depends on it stays scalar).
__device__ __forceinline__ unsigned long long rt_first_lane_u64(unsigned long long v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

// One wavefront's share of the trajectory counter and of the run's counts, in
// LDS.  Lanes take trajectories from the reserved range [next, end); when a
// pass needs more than are left, one lane reserves as many as the stopping
// lanes need, and more while many trajectories are left: a quarter of an even
// share, at most 64, of what was left when this wavefront last reserved (others
// have taken some since, so near the end it may take more than a quarter).
// Firings and end states are summed here and added to the run's counters once,
// when the wavefront ends.  With one device-wide atomic per trajectory for the
// trajectory and two for the counts, all on one line, ensembles of short
// trajectories were bound by those: the expectation and gradient of a birth-
// death process over 2^18 trajectories of 200 firings took 5.73 ms, 2.25 ms
// with the reservations and 0.84 ms with no atomic made past the last
// trajectory.
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
                // (past the last trajectory no further atomic is made)
                next = (int64_t)at + (want - left);
                end = (int64_t)at + n >= R ? INT64_MAX : (int64_t)at + n;
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

// Where a kernel's per-lane logarithms find the quick phase's table.  The
// thread and sub-wave kernels keep a copy in LDS (6 KiB per workgroup): its
// reads are counted apart from the global loads in flight, and 64 lanes'
// entries come faster than from the vector L1.  Kernels whose LDS bounds the
// network size read the constant table itself.
struct rt_log_lds_tab {
    const rt_logq* tab;
    __device__ __forceinline__ rt_logq operator()(uint32_t i) const { return tab[i]; }
};
struct rt_log_const_tab {
    __device__ __forceinline__ rt_logq operator()(uint32_t i) const { return rt_logq_const(i); }
};

template <class Tab>
struct rt_log_ctx {
    Tab tab;
    uint32_t* sc;       // RT_LOG_SCRATCH words of LDS for the accurate phase
};

template <int WAVES>
struct rt_log_lds {
    rt_logq tab[RT_LOGQ_N];
    uint32_t scratch[WAVES][RT_LOG_SCRATCH];

    // Every thread of the workgroup calls this once before the first draw.
    __device__ __forceinline__ rt_log_ctx<rt_log_lds_tab> init()
    {
        for (int i = (int)threadIdx.x; i < RT_LOGQ_N; i += (int)blockDim.x)
            tab[i] = rt_logq_const((uint32_t)i);
        __syncthreads();
        return {{tab}, scratch[threadIdx.x >> 6]};
    }
};

// The draws the quick phase left open (about one in 2^12.5): the fast phase,
// and for those it cannot certify either (one in 2^20) the accurate phase, in
// which the lanes take turns on the wave's LDS slice.  Called with the lanes
// that are open in this wavefront; true in the lanes that took the accurate
// phase.
__device__ __forceinline__ bool rt_neglog_open(uint64_t m, bool force_accurate, uint32_t* sc,
                                               double& y)
{
    int e, i;
    double z;
    rt_neglog_reduce(m, e, i, z);
    bool need = m != 0x1FFFFFFFFFFFFFull;                     // u = 1 gives +0
    y = 0.0;
    if (need && !force_accurate) {
        double yh, yl;
        rt_neglog_fast(e, i, z, yh, yl);
        y = yh;
        need = !rt_rounding_certain(yh, yl);
    }
    unsigned long long pending = __ballot(need);
    if (__builtin_expect(pending != 0ull, 0)) {
        const int me = (int)(threadIdx.x & 63u);
        while (pending) {
            const int lane = __ffsll((long long)pending) - 1;
            if (lane == me) y = rt_neglog_accurate(e, i, z, sc);
            pending &= pending - 1ull;
        }
    }
    return need;
}

// RN(-ln u) for the wave's active lanes; each lane that needs the accurate
// phase adds one to the device counter *slow and sets *took_slow (either may be
// NULL).
template <class Tab>
__device__ __forceinline__ double rt_neglog_wave(uint64_t m, bool force_accurate,
                                                 unsigned long long* slow,
                                                 const rt_log_ctx<Tab>& lc,
                                                 bool* took_slow = nullptr)
{
    double y;
    const bool open =
        !rt_neglog_quick((uint32_t)(m >> 32), (uint32_t)m, lc.tab, y) || force_accurate;
    if (took_slow) *took_slow = false;
    if (__builtin_expect(__ballot(open) != 0ull, 0)) {
        if (open) {
            const bool acc = rt_neglog_open(m, force_accurate, lc.sc, y);
            if (took_slow) *took_slow = acc;
            if (slow && acc) atomicAdd(slow, 1ull);
        }
    }
    return y;
}

// RN(-ln u) when every active lane holds the same m (a draw computed by a
// whole wavefront for one channel).  The table entry is a scalar load, which
// does not wait for the vector loads in flight; past the quick phase the value
// is computed in the first active lane and broadcast; *slow counts one per
// accurate phase.
__device__ __forceinline__ double rt_neglog_uniform(uint64_t m, unsigned long long* slow,
                                                    uint32_t* sc)
{
    double y;
    const bool open = !rt_neglog_quick(
        (uint32_t)(m >> 32), (uint32_t)m,
        [](uint32_t i) { return rt_logq_const(__builtin_amdgcn_readfirstlane(i)); }, y);
    if (__builtin_expect(__ballot(open) != 0ull, 0)) {
        const unsigned long long active = __ballot(true);
        const int first = __ffsll((long long)active) - 1;
        if ((int)(threadIdx.x & 63u) == first) {
            if (rt_neglog_open(m, false, sc, y)) atomicAdd(slow, 1ull);
        }
        y = __shfl(y, first, 64);
    }
    return y;
}

// The 53 bits behind a draw of the channel's n-th firing, from its block: the
// words' order must not be folded into the last round (the compiler would
// select that round's operands instead of its results, twice the
// instructions).
__device__ __forceinline__ uint64_t rt_block_m53(rt_u4 w, uint32_t n)
{
    asm("" : "+v"(w.x), "+v"(w.y), "+v"(w.z), "+v"(w.w));
    const uint32_t hi = (n & 1u) ? w.w : w.y, lo = (n & 1u) ? w.z : w.x;
    return ((uint64_t)(hi >> 11) << 32) | __builtin_amdgcn_alignbit(hi, lo, 11);
}

template <class Tab>
__device__ __forceinline__ double rt_exp1_wave(uint32_t k0, uint32_t k1, uint32_t traj,
                                               uint32_t net, uint32_t k, uint32_t n,
                                               unsigned long long* slow,
                                               const rt_log_ctx<Tab>& lc,
                                               bool* took_slow = nullptr)
{
    return rt_neglog_wave(rt_draw_m53(k0, k1, traj, net, k, n), false, slow, lc, took_slow);
}

// E for channel k at firing index n, computed by every active lane alike.
__device__ __forceinline__ double rt_exp1_uniform(uint32_t k0, uint32_t k1, uint32_t traj,
                                                  uint32_t net, uint32_t k, uint32_t n,
                                                  unsigned long long* slow, uint32_t* sc)
{
    return rt_neglog_uniform(rt_draw_m53(k0, k1, traj, net, k, n), slow, sc);
}
