// Alg. 1 with channels that serve by readiness (PP_SCHED_FIFO), a stage and the channel behind it per lane.
//
// Stages follow their lists, a channel takes what was ready first (equal times: the earlier in list order, which is sweep,
// then block).  Sweep by sweep, as Alg. 1's first phase deals the items out, everything a step needs is known
// although the channels' order is not: with stage n the resource r, F(m) and B(m) microbatch m's items of the channel between
// stages n and n + 1 (resource r + 1), and K = 2 (R - r),
//   * F(m + K + 1) is ready after B(m) has ended, because stage n serves B(m) before it; so before B(m) come at
//     most F(m + K), which stage n has served in the sweep after B(m)'s own, and what is before it;
//   * B(m - K + 4) is ready after F(m) has ended, because stage n + 1 serves F(m) before it; so before F(m) come at
//     most B(m - K + 3), which stage n + 1 serves in F(m)'s own sweep, and what is before it.
// Sweep t therefore goes in four steps: the stages' forward items; the channels' backward items of sweep t - 1, after
// those of the next two forward items that were ready earlier; the stages' backward items; the channels'
// forward items of sweep t, after those of the next two backward items that were ready earlier.  (Equal times: the backward item
// comes first in the second step and the forward item in the fourth, by the list.)  With positive durations this is the
// schedule of the event simulation in k_makespan_events.
//
// Left to k_makespan_events (marked MK_NOT_TAKEN), with the rest of their workgroup: zero durations, whose order within one point in
// time only the simulation defines, and times whose sum does not fit 30 bits (no schedule that
// always has an item in service is longer than the sum of all items).
//
// What bounds it: instruction issue, about 50 vector instructions per stage (with its channel) and sweep, M + 4 S - 4 sweeps.
// 40 320 plans of 8 stages, M = 64: 0.30 ms with bounds on the neighbours' next times and passes over the resources
// until every item was served, 0.05 ms now (whole call with the three other orders 321 -> 77 us).
#include "pp_makespan.h"

// A workgroup's threads, about one per resource, for the loads; half of them, a lane per stage, go on: four waves, one per
// SIMD wherever the workgroup's first lands (one wave of 256 threads with two stages per lane: 75 us of the 40 320 plans
// below, because some SIMDs got twice the waves of others).
#define FIFO_THREADS 512
#define FIFO_LATE (1 << 30)  // later than any time: an item that is not there, or served

__device__ __forceinline__ int fifo_max(int a, int b) { return a > b ? a : b; }

// A stage, and the channel to the next one.
struct fifo_pair {
    int idle, df, db;        // the stage: when it is idle, its durations
    int free, cf, cb;        // the channel
    // When the channel's next items were ready: the forward ones of this sweep and the next, the backward ones of the sweep
    // before, this and the next; and their ends, where they have been served.
    int f1, f2, g0, g1, g2, endF1, endF2, endB0, endB1, endB2;
    // The sweeps since the stage's first forward and backward item (as unsigned numbers: M or more is none).  The last stage's
    // merged items are its forward ones, and end again as backward ones that take no time.
    unsigned tf, tb;
};

// Serves the channel's item that was ready at `at`, where `when`.
__device__ __forceinline__ void fifo_serve(fifo_pair &s, bool when, int &at, int duration, int &end) {
    const int done = fifo_max(s.free, at) + duration;
    s.free = when ? done : s.free;
    end = when ? done : end;
    at = when ? FIFO_LATE : at;
}

// LG = a.lanes_per lanes per candidate (a power of two, at least S), lane q holds stage q.
__global__ __launch_bounds__(FIFO_THREADS) void k_makespan_fifo(mk_args a) {
    extern __shared__ int lds[];
    const int S = a.S, L = a.L, D = a.D, M = a.Ms[0], LG = a.lanes_per, SP = S | 1;
    const int R = 2 * S - 1, J = 2 * R - 1;
    const int tid = threadIdx.x, per = a.groups;  // candidates per workgroup
    int *so = lds, *sb = so + per * SP, *sf = sb + per * SP;
    const long long c0 = a.first + (long long)blockIdx.x * per;
    for (int t = tid; t < per * S; t += blockDim.x) {
        const int i = t / S, n = t - i * S;
        const long long c = c0 + i;
        int o = 0, e = 0;
        if (c < a.N) {
            if (a.orderings) o = a.orderings[c * S + n];
            e = a.bounds[c * S + n];
        }
        so[i * SP + n] = o;
        sb[i * SP + n] = e;
    }
    __syncthreads();
    if (tid < per) sf[tid] = c0 + tid < a.N ? mk_check_rows(a, c0 + tid, so + tid * SP, sb + tid * SP) : 0;
    __syncthreads();
    if (tid >= per * LG) return;
    const int i = tid / LG, q = tid - i * LG;
    const long long c = c0 + i;
    const bool live = c < a.N;
    const int fault = sf[i];
    const bool ok = live && !fault;
    fifo_pair s;
    bool zero = false;
    long long x = 0, y = 0, cx = 0, cy = 0;
    const bool there = ok && q < S;
    s.tf = there ? (unsigned)(-2 * q) : 1u << 31;
    s.tb = !there ? 1u << 31 : q == S - 1 ? s.tf : (unsigned)(2 * q + 2 - 2 * R);
    if (there) {
        const int *o = so + i * SP, *e = sb + i * SP;
        const int e1 = e[q], e0 = q ? e[q - 1] : 0;
        x = a.PF[e1] - a.PF[e0];
        y = a.PB[e1] - a.PB[e0];
        if (q == S - 1) { x += y; y = 0; }
        zero |= x <= 0;
        if (q < S - 1) {
            const size_t at = ((size_t)o[q] * D + o[q + 1]) * L + (size_t)(e1 - 1);
            cx = a.XF[at];
            cy = a.XB[at];
            zero |= y <= 0 || cx <= 0 || cy <= 0;
        }
    }
    s.df = (int)x;
    s.db = (int)y;
    s.cf = (int)cx;
    s.cb = (int)cy;
    // (anything at 2^30 or above is out already: the sum of at most 126 such cannot overflow)
    const long long cap = PP_TIME_CAP;
    long long sum = (x < cap ? x : cap) + (y < cap ? y : cap) + (cx < cap ? cx : cap) + (cy < cap ? cy : cap);
    s.idle = s.free = 0;
    s.f1 = s.f2 = s.g0 = s.g1 = s.g2 = FIFO_LATE;
    s.endF1 = s.endF2 = s.endB0 = s.endB1 = s.endB2 = 0;
    int odd = zero;
    for (int off = 1; off < LG; off <<= 1) {
        sum += __shfl_xor(sum, off);
        odd |= __shfl_xor(odd, off);
    }
    // (the workgroup's candidates are taken or left together: k_makespan_events simulates whole waves
    // of neighbours wherever one of them is left.  All four schedules, a seventh of the cuts with nothing to
    // send, 10^6 plans of 2 stages, M = 32: 1.95 ms plan by plan, 1.15 together, 1.19 in that kernel alone)
    const bool taken = __syncthreads_and(!ok || (!odd && sum <= (long long)PP_TIME_CAP / M));
    // (a sweep more than there are serves nothing, nor does a channel behind the last stage hand anything on)
    const bool first = q == 0, reaches = q + 1 < LG;
    // (a wave without a plan has nothing to sweep; one that has one has items of positive length, so M is below 2^30)
    const int sweeps = taken && __ballot(ok) ? M + J - 1 : 0;
    for (int t = 0; t < sweeps; t += 2) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            // the stage's forward item, which the channel before has let go in the last sweep
            int from = __builtin_amdgcn_update_dpp(0, s.endF1, DPP_WAVE_SHR1, 0xf, 0xf, false);
            from = first ? 0 : from;
            int end = fifo_max(s.idle, from) + s.df;
            bool here = s.tf++ < (unsigned)M;
            s.idle = here ? end : s.idle;
            // (what was the next sweep's item is this one's; the new one is ready now)
            s.endF1 = s.endF2;
            s.f1 = s.f2;
            s.f2 = here ? end : FIFO_LATE;
            // the channel's backward item of the sweep before
            const int g = s.g0;
            bool due = g < FIFO_LATE;
            fifo_serve(s, due & (s.f1 < g), s.f1, s.cf, s.endF1);
            fifo_serve(s, due & (s.f2 < g), s.f2, s.cf, s.endF2);
            fifo_serve(s, due, s.g0, s.cb, s.endB0);
            // the stage's backward item, ready for the channel before it
            end = fifo_max(s.idle, s.endB0) + s.db;
            here = s.tb++ < (unsigned)M;
            s.idle = here ? end : s.idle;
            const int ready = here ? end : FIFO_LATE;
            const int right = __builtin_amdgcn_update_dpp(0, ready, DPP_WAVE_SHL1, 0xf, 0xf, false);
            s.g2 = reaches ? right : FIFO_LATE;
            // the channel's forward item of this sweep
            const int f = s.f1;
            due = f < FIFO_LATE;
            fifo_serve(s, due & (s.g1 < f), s.g1, s.cb, s.endB1);
            fifo_serve(s, due & (s.g2 < f), s.g2, s.cb, s.endB2);
            fifo_serve(s, due, s.f1, s.cf, s.endF1);
            s.g0 = s.g1;
            s.endB0 = s.endB1;
            s.g1 = s.g2;
            s.endB1 = s.endB2;
        }
    }
    if (live && q == 0) {
        if (fault) pp_raise(a.status, fault);
        a.T_out[c] = fault ? PP_INF64 : (taken ? (long long)s.idle : MK_NOT_TAKEN);
    }
}

int pp_launch_makespan_fifo(const mk_args &a, hipStream_t st) {
    const int R = 2 * a.S - 1;
    if (R > 64) return PP_ERR_INVALID_ARG;
    mk_args b = a;
    int each = 1;  // (threads per candidate: its resources, rounded up to a power of two)
    while (each < R) each <<= 1;
    b.lanes_per = each > 1 ? each / 2 : 1;
    const int per = b.groups = FIFO_THREADS / each, threads = per * each;
    const size_t lds = (size_t)per * (2 * (a.S | 1) + 1) * 4;
    // A launch has fewer than 2^32 threads.  At up to 64 threads per candidate that is fewer candidates than
    // a list may hold (all 12! orderings, 32 each), so long lists take several launches.
    const long long groups = (a.N + per - 1) / per, most = ((1ll << 32) - 1) / threads;
    for (long long g = 0; g < groups; g += most) {
        b.first = g * per;
        hipLaunchKernelGGL(k_makespan_fifo, dim3((unsigned)(groups - g < most ? groups - g : most)), dim3(threads), lds, st, b);
        if (hipGetLastError() != hipSuccess) return PP_ERR_HIP;
    }
    return PP_OK;
}
