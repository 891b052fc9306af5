// T of a plan without running its schedule: the longest path through the schedule, in closed form.
//
// Alg. 1's schedule (pp_makespan.hip) is a max-plus recurrence, so T is the longest path from the first item to
// the last in the graph whose arcs are "the same microbatch's next block" and "the resource's next item".  Resources
// r = 1..R, a_r and b_r the durations of their forward and backward blocks (the last one's merged block: a_R,
// b_R = 0), c_r = a_r + b_r.  A walk along the path in sweeps: a sweep spent at resource r gains c_r where the walk
// stays (one item of each side), a_r where it passes upwards, b_r where it passes downwards; before the resource's first
// backward item (sweep 2R - r) staying gains a_r alone, after its last forward item (sweep r + M - 1) b_r alone.
// All walks take M + 2R - 2 sweeps.
//   * Every cycle (up from r to r', back down, and on) gains at most max c over its resources a sweep.  So a walk
//     is no longer than one that spends all it can at a single resource r, and goes everywhere else directly.
//   * Before resource r is reached, and after it is left, time can be spent where a (or b) is largest, but
//     only in the sweeps in which the peak p of the way there has no backward item yet: 2 (R - p) of them.
// With sums Sa(p), Sb(p) and largest values A(p), B(p) over the resources 1..p, and K = 2 (R - p):
//     up(p) = Sa(p) + Sb(p) + K A(p),   down(p) = Sa(p) + Sb(p) + K B(p),
//     T = max over r of c_r (M - 2 (R - r) - 2) - Sa(r-1) - Sb(r-1) + max_{p >= r} up(p) + max_{p >= r} down(p)
// over the resources with 2 (R - r) <= M - 2.  In a pipeline that does not fill (M < 2R) the walk may also
// spend no sweep at any resource while both of its sides are served: for every peak p, with k = min(K, M - 1),
//     Sa(p) + Sb(p) + k A(p) + (M - 1) B(p)   and   Sa(p) + Sb(p) + (M - 1) A(p) + k B(p).
// Where a resource's two sides do not wait for each other (full-duplex channels) it is no r and no p, and the
// second kind counts for every M.  All terms are walks, so none is longer than T, and every value on the way is
// below the bound of Lemma 1 on T; sums of V are taken without regard to overflow, which the caller rules out.
//
// One pass over the resources keeps, for every microbatch count, the largest of the first term alone, with
// `up`, with `down` and with both so far: O(S) instructions per plan instead of O(M S).
#pragma once

#include "pp_makespan.h"

template <typename V> struct mk_unsigned;
template <> struct mk_unsigned<int> { typedef unsigned type; };
template <> struct mk_unsigned<long long> { typedef unsigned long long type; };

template <typename V> __device__ __forceinline__ V mk_sum(V x, V y) {
    typedef typename mk_unsigned<V>::type U;
    return (V)((U)x + (U)y);
}
template <typename V> __device__ __forceinline__ V mk_less(V x, V y) {
    typedef typename mk_unsigned<V>::type U;
    return (V)((U)x - (U)y);
}
__device__ __forceinline__ long long mk_times(long long x, int k) {
    return (long long)((unsigned long long)x * (unsigned long long)k);
}
// (V = int is for times and counts below 2^24, which pp_time_limit sees to: the product is one full-rate instruction)
__device__ __forceinline__ int mk_times(int x, int k) { return (int)(((unsigned)x & 0xffffff) * ((unsigned)k & 0xffffff)); }
template <typename V> __device__ __forceinline__ V mk_larger(V x, V y) { return x > y ? x : y; }

// The walks through the resources so far, for NM microbatch counts.
template <typename V, int NM>
struct mk_path {
    V sum, A, B;  // Sa + Sb, A, B
    V at[NM], up[NM], down[NM], both[NM], brief[NM];

    __device__ __forceinline__ void start() {
        constexpr V lowest = (V)((V)1 << (sizeof(V) * 8 - 2)) * -2;
        sum = A = B = 0;
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            at[q] = up[q] = down[q] = both[q] = lowest;
            brief[q] = 0;
        }
    }
    // The next resource: K = 2 (resources behind it).  turn: its two sides wait for each other.  briefly: walks
    // of the second kind count (2 bits per count would do; the counts are uniform, and so are the branches).
    __device__ __forceinline__ void step(V a, V b, int K, bool turn, const int (&M)[NM], const bool (&briefly)[NM]) {
        const V before = sum;
        sum = mk_sum(mk_sum(sum, a), b);
        A = mk_larger(A, a);
        B = mk_larger(B, b);
        if (!turn) return;
        const V c = mk_sum(a, b), u = mk_sum(sum, mk_times(A, K)), d = mk_sum(sum, mk_times(B, K));
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            if (M[q] - 2 >= K) {
                at[q] = mk_larger(at[q], mk_less(mk_times(c, M[q] - 2 - K), before));
                up[q] = mk_larger(up[q], mk_sum(at[q], u));
                down[q] = mk_larger(down[q], mk_sum(at[q], d));
                both[q] = mk_larger(both[q], mk_larger(mk_sum(up[q], d), mk_sum(down[q], u)));
            }
            if (briefly[q]) {
                const int m = M[q] - 1, k = K < m ? K : m;
                const V x = mk_sum(mk_sum(sum, mk_times(A, k)), mk_times(B, m));
                const V y = mk_sum(mk_sum(sum, mk_times(A, m)), mk_times(B, k));
                brief[q] = mk_larger(brief[q], mk_larger(x, y));
            }
        }
    }
    __device__ __forceinline__ V longest(int q) const { return mk_larger(both[q], brief[q]); }
};

// ---------------------------------------------------------------- plans in memory, one per lane

#define MK_COUNTS 4         // microbatch counts a lane works on at once; more counts: blockIdx.y
#define MK_PATH_WAVES 8     // most waves per workgroup
#define MK_PATH_GRID 2048   // most workgroups; they go round
#define MK_AT_ONCE 4        // stages whose transfer times a lane asks for together
#define MK_SPREAD 4096
#define MK_PICK_WAVES 4      // short lists of up to so many groups of 64: one workgroup schedules and picks

// LDS: PF and PB in pairs, then per wave one word per stage of each of its 64 plans, in rows an odd number
// of words apart: the device (0xffff: none such), and above it the stage's bound (none such: L and the sign bit).
__host__ __device__ static inline size_t mk_path_table_bytes(int L) { return (size_t)(L + 1) * 16; }
// (of the planner's own plans, whose times are known to fit, the low halves)
__host__ __device__ static inline size_t mk_known_table_bytes(int L) { return ((size_t)(L + 2) * 8) & ~(size_t)15; }
__host__ __device__ static inline size_t mk_path_wave_bytes(int S) { return (size_t)64 * (S | 1) * 4; }

// Device n of the orderings with lexicographic rank c < 12!: dig holds their digits, 4 bits each.
__device__ __forceinline__ unsigned long long mk_rank_digits(int D, unsigned c) {
    unsigned long long dig = 0;
#pragma unroll
    for (unsigned k = 1; k <= 12; ++k)
        if ((int)k <= D) {
            dig |= (unsigned long long)(c % k) << (4 * (D - (int)k));
            c /= k;
        }
    return dig;
}

// What a lane finds out about its plan.
struct mk_plan_info {
    int fault;
    bool fits;        // (32 bits) no sum of the call leaves them
    long long worst;  // (64 bits) the largest per-resource time
};

// The steps of stage n of xi through the walks: its own times, and those of the link into it.
template <int MODE, int NM, typename V>
__device__ __forceinline__ void mk_stage(mk_path<V, NM> &path, int n, int xi, V F, V B, V cf, V cb, const int (&M)[NM],
                                         const bool (&briefly)[NM]) {
    const bool last = n == xi - 1;
    if (MODE == PP_SCHED_ADDITIVE) {
        // the transfers over a stage's inbound link are part of its passes
        const V f = mk_sum(F, cf), b = mk_sum(B, cb);
        path.step(last ? mk_sum(f, b) : f, last ? (V)0 : b, 2 * (xi - 1 - n), true, M, briefly);
    } else if (MODE == PP_SCHED_GPIPE) {
        path.step(cf, cb, 0, false, M, briefly);
        path.step(F, B, 0, false, M, briefly);
    } else {
        const int K = 4 * (xi - 1 - n);
        if (n) path.step(cf, cb, K + 2, MODE != PP_SCHED_DUPLEX, M, briefly);
        path.step(last ? mk_sum(F, B) : F, last ? (V)0 : B, K, true, M, briefly);
    }
}
template <int MODE, int NM, typename V>
__device__ __forceinline__ V mk_result(const mk_path<V, NM> &path, int q, int M) {
    // (GPipe's order: two flow shops of M equal jobs, one after the other.  A and B, of different resources maybe, fit 24 bits
    // each and their sum may not.)
    if (MODE == PP_SCHED_GPIPE) return mk_sum(path.sum, mk_sum(mk_times(path.A, M - 1), mk_times(path.B, M - 1)));
    return path.longest(q);
}
template <int MODE, int NM>
__device__ __forceinline__ void mk_briefly(const int (&M)[NM], int xi, bool (&briefly)[NM]) {
    const int R = MODE == PP_SCHED_ADDITIVE ? xi : 2 * xi - 1;
#pragma unroll
    for (int q = 0; q < NM; ++q) briefly[q] = MODE == PP_SCHED_DUPLEX || M[q] < 2 * R;
}

// Looks at a plan's rows stage by stage.
struct mk_row_check {
    unsigned long long seen;
    int e0;
    bool bad, torn;
    __device__ __forceinline__ void start() { seen = 0; e0 = 0; bad = torn = false; }
    __device__ __forceinline__ void stage(const mk_args &a, const int *row, int n, int w) {
        const int o = w & 0xffff, e = (int)((unsigned)w >> 16);
        bad |= o >= a.D;
        if (a.D <= 64) {
            bad |= (seen >> (o & 63)) & 1;
            seen |= 1ull << (o & 63);
        } else if (a.orderings) {
            for (int i = 0; i < n; ++i) bad |= (row[i] & 0xffff) == o;
        }
        torn |= e <= e0 || e > a.L;
        e0 = e;
    }
    // (a bad ordering is reported alone: its plan is not looked at)
    __device__ __forceinline__ int fault(const mk_args &a, bool live) const {
        return !live ? 0 : bad ? PP_FAULT_ORDERING : torn || e0 != a.L ? PP_FAULT_BOUNDS : 0;
    }
};

// Where the times of the link between two stages lie (words of the stages; 0, which is always there, if one is no good).
__device__ __forceinline__ size_t mk_link_at(const mk_args &a, int before, int w, bool live) {
    const int o = w & 0xffff, o0 = before & 0xffff, e0 = (int)((unsigned)before >> 16);
    const bool there = o < a.D && o0 < a.D && e0 >= 1 && e0 <= a.L && live;
    // (D <= 2^10, L <= 2^11)
    const unsigned link = (unsigned)mk_times(o0, a.D) + (unsigned)o;
    return there ? (size_t)((link & 0xffffff) * ((unsigned)a.L & 0xffffff) + (unsigned)(e0 - 1)) : 0;
}

// The plan of xi stages in the wave's rows, of this lane (live: there is one), in 32-bit sums.  PT: pairs (PF, PB).
// The transfer times of the next stages are on their way while these are looked at.  (In registers: with a column of LDS
// per lane instead, and the stages in a loop of their own, fewer waves fit a compute unit: 58 -> 87 us for 131 071 plans
// of 32 stages.)
template <int MODE, int NM>
__device__ __forceinline__ mk_plan_info mk_plan32(const mk_args &a, const int *row, const long long *PT, int xi,
                                                  bool live, const int (&M)[NM], int limit, long long (&T)[NM]) {
    mk_path<int, NM> path;
    path.start();
    bool briefly[NM];
    mk_briefly<MODE>(M, xi, briefly);
    struct piece { long long f[MK_AT_ONCE], b[MK_AT_ONCE]; int w[MK_AT_ONCE]; };
    // (`before`: the word of the stage before)
    auto ask = [&](piece &x, int n0, int before) {
#pragma unroll
        for (int u = 0; u < MK_AT_ONCE; ++u) {
            const int n = n0 + u;
            x.f[u] = x.b[u] = 0;
            x.w[u] = before;
            if (n >= xi) continue;
            const int w = row[n];
            const size_t at = mk_link_at(a, before, w, live);
            x.w[u] = before = w;
            if (n) { x.f[u] = a.XF[at]; x.b[u] = a.XB[at]; }
        }
        return before;
    };
    piece now, then;
    int asked = ask(now, 0, 0);
    mk_row_check check;
    check.start();
    int f0 = (int)PT[0], b0 = (int)PT[1];
    long long p0 = PT[0] + PT[1], over = 0;
    unsigned most = 0;
    for (int n0 = 0; n0 < xi; n0 += MK_AT_ONCE) {
        if (n0 + MK_AT_ONCE < xi) asked = ask(then, n0 + MK_AT_ONCE, asked);
#pragma unroll
        for (int u = 0; u < MK_AT_ONCE; ++u) {
            const int n = n0 + u;
            if (n >= xi) continue;
            const int w = now.w[u], e1 = (int)((unsigned)w >> 16), e = e1 <= a.L ? e1 : a.L;
            check.stage(a, row, n, w);
            const long long pf = PT[2 * e], pb = PT[2 * e + 1], p = pf + pb, x = now.f[u] + now.b[u];
            const int F = mk_less((int)pf, f0), B = mk_less((int)pb, b0);
            f0 = (int)pf;
            b0 = (int)pb;
            // (sums of two non-negative times: what is 31 bits or less is so in its parts)
            over |= (p - p0) | x;
            const unsigned s = (unsigned)(p - p0);
            p0 = p;
            if (MODE == PP_SCHED_ADDITIVE) {
                const unsigned both = s + (unsigned)x;  // (of two numbers below 2^31, or over is set)
                over |= (long long)(both & 0x80000000u) << 1;
                most = most > both ? most : both;
            } else {
                most = most > s ? most : s;
                most = most > (unsigned)x ? most : (unsigned)x;
            }
            mk_stage<MODE>(path, n, xi, F, B, (int)now.f[u], (int)now.b[u], M, briefly);
        }
        now = then;
    }
#pragma unroll
    for (int q = 0; q < NM; ++q) T[q] = mk_result<MODE>(path, q, M[q]);
    mk_plan_info i;
    i.fault = check.fault(a, live);
    i.worst = 0;
    i.fits = !live || i.fault || (!(over >> 31) && limit >= 0 && most <= (unsigned)limit);
    return i;
}

// The same of a plan whose largest time is known to fit (its C), of valid devices: nothing is checked, and of every number
// the low half is read.  What it returns is negative if one of the bounds is none (it is taken for L).
template <int NM>
__device__ __forceinline__ int mk_plan_known(const mk_args &a, const int *row, const int2 *PT, int xi, bool good,
                                             const int (&M)[NM], long long (&T)[NM]) {
    mk_path<int, NM> path;
    path.start();
    bool briefly[NM];
    mk_briefly<PP_SCHED_PE>(M, xi, briefly);
    const int *XF = (const int *)a.XF, *XB = (const int *)a.XB;
    struct piece { int f[MK_AT_ONCE], b[MK_AT_ONCE], e[MK_AT_ONCE]; };
    int before = 0, cut = 0, all = 0;  // the device and the bound of the stage before; the words together
    auto ask = [&](piece &x, int n0) {
#pragma unroll
        for (int u = 0; u < MK_AT_ONCE; ++u) {
            const int n = n0 + u;
            x.f[u] = x.b[u] = x.e[u] = 0;
            if (n >= xi) continue;
            const int w = row[n];
            const unsigned link = (unsigned)mk_times(before, a.D) + (unsigned)(w & 0xffff);
            const size_t at = good ? (size_t)((link & 0xffffff) * ((unsigned)a.L & 0xffffff) + (unsigned)cut - 1) * 2 : 0;
            if (n) { x.f[u] = XF[at]; x.b[u] = XB[at]; }
            all |= w;
            before = w & 0xffff;
            cut = x.e[u] = good ? w >> 16 & 0x7fff : 0;
        }
    };
    piece now, then;
    ask(now, 0);
    int2 p = PT[0];
    for (int n0 = 0; n0 < xi; n0 += MK_AT_ONCE) {
        if (n0 + MK_AT_ONCE < xi) ask(then, n0 + MK_AT_ONCE);
#pragma unroll
        for (int u = 0; u < MK_AT_ONCE; ++u) {
            const int n = n0 + u;
            if (n >= xi) continue;
            const int2 q = PT[now.e[u]];
            mk_stage<PP_SCHED_PE>(path, n, xi, mk_less(q.x, p.x), mk_less(q.y, p.y), now.f[u], now.b[u], M, briefly);
            p = q;
        }
        now = then;
    }
#pragma unroll
    for (int q = 0; q < NM; ++q) T[q] = path.longest(q);
    return good ? all : 0;
}

// In 64 bits.
template <int MODE, int NM>
__device__ __forceinline__ mk_plan_info mk_plan64(const mk_args &a, const int *row, int xi, bool live, const int (&M)[NM], long long (&T)[NM]) {
    mk_path<long long, NM> path;
    path.start();
    bool briefly[NM];
    mk_briefly<MODE>(M, xi, briefly);
    mk_row_check check;
    check.start();
    long long f0 = a.PF[0], b0 = a.PB[0], worst = 0;
    int before = 0;
#pragma unroll 1
    for (int n = 0; n < xi; ++n) {
        const int w = row[n], e1 = (int)((unsigned)w >> 16), e = e1 <= a.L ? e1 : a.L;
        const size_t at = mk_link_at(a, before, w, live);
        const long long cf = n ? a.XF[at] : 0, cb = n ? a.XB[at] : 0;
        check.stage(a, row, n, w);
        before = w;
        const long long pf = a.PF[e], pb = a.PB[e], F = pf - f0, B = pb - b0;
        f0 = pf;
        b0 = pb;
        worst = mk_larger(worst, mk_larger(F + B, cf + cb));
        mk_stage<MODE>(path, n, xi, F, B, cf, cb, M, briefly);
    }
#pragma unroll
    for (int q = 0; q < NM; ++q) T[q] = mk_result<MODE>(path, q, M[q]);
    mk_plan_info i;
    i.fault = check.fault(a, live);
    i.worst = worst;
    i.fits = true;
    return i;
}

// The smallest T of each of the workgroup's waves to the workgroup's partials, or, where the launch is one
// workgroup, the winners' records (lds: a pair per wave and count; bounds and C are where write_winner reads them).
template <int NM>
__device__ __forceinline__ void mk_leave_least(const mk_args &a, const tc_pair (&least)[NM], tc_pair *lds) {
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    tc_pair w[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) w[q] = wave_tc_min(least[q]);
    if (waves > 1 || a.pick_here) {
        __syncthreads();  // what lies in the LDS has been read
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < NM; ++q) lds[wave * NM + q] = w[q];
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        const int slot = (int)blockIdx.y * NM + q;
        if (slot >= a.nM || wave != q % waves) continue;
        tc_pair v = w[q];
        if (waves > 1)
            for (int o = 0; o < waves; ++o) v = tc_min(v, lds[o * NM + q]);
        if (a.pick_here) write_winner(a, slot, v, lane);
        else if (lane == 0) a.part[(long long)slot * gridDim.x + blockIdx.x] = v;
    }
}

// The workgroup's microbatch counts (1 where there are fewer).  Selected with constant indices: a run-time index
// into the argument struct can make the compiler keep a copy of all of it in scratch memory.
template <int NM>
__device__ __forceinline__ void mk_counts(const mk_args &a, int (&M)[NM]) {
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        M[q] = 1;
#pragma unroll
        for (int i = 0; i < PP_MAX_M_LIST; ++i) M[q] = i == (int)blockIdx.y * NM + q ? a.Ms[i] : M[q];
    }
}

// A workgroup's waves take groups of 64 plans; with a.search all plans of 1 .. a.search stages of the group's
// candidates, each wave some of the stage counts.  KNOWN: the plans are those the partition program has left (MODE is
// PP_SCHED_PE): no time of one is longer than its C, and a bad ordering's C is PP_INF64.  FREE: k_band_free may have scheduled
// some of them.
template <int MODE, int NM, bool KNOWN, bool FREE = false>
__device__ __forceinline__ void mk_path_body(const mk_args &a) {
    extern __shared__ __align__(16) int rows[];
    const int tid = threadIdx.x, lane = tid & 63, threads = blockDim.x, waves = threads >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S, L = a.L, D = a.D;
    long long *PT = (long long *)rows;
    int2 *PK = (int2 *)rows;
    // (one trip to memory for what the header says)
    const unsigned active = a.rlist ? a.hdr->share_active : 0, nreps = a.rlist ? a.hdr->share_nreps : 0;
    const bool listed = active;
    const long long todo = listed ? nreps : a.N, groups = (todo + 63) / 64;
    const bool has_free = FREE && mk_has_free(a);
    const int counts = a.search ? a.search : 1, per = a.search ? 1 : waves;
    tc_pair least[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) least[q] = {PP_INF64, INT64_MAX};
    // (a workgroup without a group of its own needs no tables)
    bool idle = (long long)blockIdx.x * per >= groups;
    if (FREE && has_free) {
        idle = true;
        // (of the plans that are scheduled already, a minimum per 64 candidates; where they are all of this workgroup's, it
        // needs no tables: 2^20 candidates of 32 stages, the T of each read instead and the tables always: 15.0, so 10.6 us)
        for (long long i = tid; i < groups; i += threads) {
            const long long g = (i / waves * gridDim.x + blockIdx.x) * waves + i % waves;
            if (g >= groups) break;
            idle = idle && a.free_bits[g] == ~0ull >> (todo - g * 64 < 64 ? 64 - (todo - g * 64) : 0);
        }
        for (long long g = (long long)blockIdx.x * threads + tid; g < groups; g += (long long)gridDim.x * threads)
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int slot = (int)blockIdx.y * NM + q;
                const long long v = slot < a.nM ? a.free_least[slot * groups + g] : -1;
                if (v >= 0) least[q] = tc_min(least[q], {v >> 6, g * 64 + (v & 63)});
            }
        idle = __syncthreads_and(idle);
    }
    auto table = [&](int i, long long f, long long b) {
        if (KNOWN) {
            PK[i] = make_int2((int)f, (int)b);
        } else {
            PT[2 * i] = f;
            PT[2 * i + 1] = b;
        }
    };
    if (L < 4 * threads) {
        for (int i = idle ? L + 1 : tid; i <= L; i += threads) table(i, a.PF[i], a.PB[i]);
    } else {
        // (of many layers 16 loads in flight: 2000 plans of 8 stages, 2000 layers, a wave to a workgroup, three counts 29.6 us for the
        // call with two, 24.3 so; of few, more code to fetch: the plans of every stage count of 8!, 128 layers 28.6 and 29.4)
        for (int i0 = idle ? L + 1 : tid; i0 <= L; i0 += 8 * threads) {
            long long f[8], b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * threads <= L ? i0 + u * threads : L;
                f[u] = a.PF[i];
                b[u] = a.PB[i];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * threads <= L) table(i0 + u * threads, f[u], b[u]);
        }
    }
    int *mine = rows + (KNOWN ? mk_known_table_bytes(L) : mk_path_table_bytes(L)) / 4 + wave * (mk_path_wave_bytes(S) / 4);
    int M[NM], mmax = 1;
    mk_counts<NM>(a, M);
#pragma unroll
    for (int q = 0; q < NM; ++q) mmax = M[q] > mmax ? M[q] : mmax;
    __syncthreads();
    for (long long g = idle ? groups : (long long)blockIdx.x * per + (a.search ? 0 : wave); g < groups; g += (long long)gridDim.x * per) {
        const long long at = g * 64 + lane;
        const bool live = at < todo;
        const long long c = !live ? 0 : listed ? pp_share_at(a.hdr, a.rlist, a.N, at) : at;
        const int held = (int)(todo - g * 64 < 64 ? todo - g * 64 : 64);  // plans of this group
        const unsigned long long ended = FREE && has_free ? a.free_bits[g] : 0;
        const bool done = FREE && (ended >> lane & 1);
        if (FREE && ended && !__ballot(live && !done)) continue;
        // (every other round of stage counts backwards: the waves' shares are alike)
        for (int turn = 0; turn * waves < counts || !a.search; ++turn) {
            const int k = turn * waves + (turn & 1 ? waves - 1 - wave : wave);
            const int xi = a.search ? k + 1 : S, SP = xi | 1;
            if (a.search && xi > counts) continue;
            const int bnd_off = a.search ? xi * (xi - 1) / 2 : a.bnd_off;
            const int limit = pp_time_limit(MODE == PP_SCHED_GPIPE ? 2ll * mmax + 4 * xi : mmax, xi);
            const long long C = KNOWN && live ? a.C[c * counts + (a.search ? xi - 1 : 0)] : 0;
            // the group's rows, entry by entry: as many loads in flight as there are stages, up to 8
            const int di = 64 / xi, dn = 64 - di * xi;
            int i = lane / xi, n = lane - i * xi;
            __builtin_amdgcn_wave_barrier();
            for (int t0 = 0; t0 < xi; t0 += 8) {
                int o[8], e[8], to[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const long long ci = listed ? (long long)__shfl((int)c, i & 63) : g * 64 + i;
                    to[u] = t0 + u < xi && i < held ? i * SP + n : -1;
                    o[u] = to[u] >= 0 && a.orderings ? a.orderings[ci * a.ord_stride + n] : 0;
                    e[u] = to[u] >= 0 ? a.bounds[ci * a.bnd_stride + bnd_off + n] : 0;
                    n += dn;
                    i += di;
                    if (n >= xi) { n -= xi; ++i; }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (to[u] >= 0)
                        mine[to[u]] = (o[u] >= 0 && o[u] < D ? o[u] : 0xffff) |
                                      (int)((unsigned)(e[u] >= 1 && e[u] <= L ? e[u] : 0x8000 | L) << 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int *row = mine + lane * SP;
            if (!KNOWN && !a.orderings && live) {
                // the list of all D! orderings: device n is the digit-th of those left
                if (D <= 12) {
                    unsigned long long left = 0xBA9876543210ull;
                    const unsigned long long dig = mk_rank_digits(D, (unsigned)c);
                    for (int m = 0; m < xi; ++m) {
                        const int d4 = (int)(dig >> (4 * m) & 15) * 4;
                        const unsigned long long low = (1ull << d4) - 1;
                        row[m] = (row[m] & (int)0xffff0000) | (int)(left >> d4 & 15);
                        left = (left & low) | (left >> 4 & ~low);
                    }
                } else {
                    unsigned long long rem = (unsigned long long)c;
                    unsigned used = 0;
                    for (int m = 0; m < xi; ++m) row[m] = (row[m] & (int)0xffff0000) | pp_unrank_next(D, m, rem, used);
                }
            }
            long long T[NM];
            mk_plan_info p = {};
            if (KNOWN) {
                // (the rows of a wave are looked at only where one of its orderings is bad, whose C says so, or a bound is none)
                const bool bad = C == PP_INF64 && !done;
                const int all = mk_plan_known<NM>(a, row, PK, xi, live && !bad && !done, M, T);
                if (__ballot(bad || all < 0)) {
                    mk_row_check check;
                    check.start();
                    for (int n = 0; n < xi; ++n) check.stage(a, row, n, row[n]);
                    p.fault = check.fault(a, live && !done);
                }
                p.fits = !live || done || p.fault || C <= limit;
            } else {
                p = mk_plan32<MODE, NM>(a, row, PT, xi, live, M, limit, T);
            }
            if (__ballot(!p.fits)) p = mk_plan64<MODE, NM>(a, row, xi, live && !done, M, T);
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int slot = (int)blockIdx.y * NM + q;
                if (slot >= a.nM || !live || (FREE && done)) continue;
                // (what the 32-bit sums took has no time that long)
                const int fault = p.fault ? p.fault : p.worst ? overflow_fault(p.worst, M[q], xi) : 0;
                if (fault) { T[q] = PP_INF64; pp_raise(a.status, fault); }
                if (a.T_out) a.T_out[((long long)slot * a.N + c) * a.t_stride + (a.search ? xi - 1 : a.t_off)] = T[q];
                if (a.part) least[q] = tc_min(least[q], {T[q], a.search ? c * a.search + xi - 1 : c});
            }
            if (!a.search) break;
        }
    }
    if (a.part) mk_leave_least(a, least, (tc_pair *)rows);
}

// The launch of mk_path_body: workgroups, waves in each, counts per lane, LDS, and whether the one workgroup picks the
// winners.
struct mk_path_launch { unsigned grid; int waves, counts; size_t lds; int pick; };

static inline mk_path_launch mk_path_shape(const mk_args &a) {
    mk_path_launch l;
    const size_t table = a.hdr ? mk_known_table_bytes(a.L) : mk_path_table_bytes(a.L), each = mk_path_wave_bytes(a.S);
    int most = (int)((64 * 1024 - table) / each);
    most = most < MK_PATH_WAVES ? most : MK_PATH_WAVES;
    const long long groups = (a.N + 63) / 64;
    // Plans worked out from LDS: up to MK_SPREAD waves in all, the counts of a call go to different workgroups (blockIdx.y), each
    // of which works the plans out for itself, because there are SIMDs without a wave otherwise (8! orderings, four counts
    // 16.6 -> 14.4 us).  Not plans from memory: 131 071 of 32 stages, two counts 58 -> 105 us.
    l.counts = a.nM == 1 || (a.fuse && groups * a.nM <= MK_SPREAD) ? 1 : a.nM == 2 ? 2 : MK_COUNTS;
    l.pick = 0;
    if (a.search) {
        l.waves = a.search < most ? a.search : most;
        l.pick = a.part && groups == 1;
        l.grid = (unsigned)(groups < MK_PATH_GRID ? groups : MK_PATH_GRID);
    } else {
        // short lists: one workgroup that picks too; longer ones: a workgroup per compute unit first
        l.pick = a.part && groups <= most && groups <= MK_PICK_WAVES;
        const long long want = l.pick ? groups : (groups + 255) / 256;
        l.waves = (int)(want < 1 ? 1 : want < 4 || l.pick ? want : 4);
        l.waves = l.waves < most ? l.waves : most;
        const long long grid = (groups + l.waves - 1) / l.waves;
        l.grid = (unsigned)(grid < MK_PATH_GRID ? grid : MK_PATH_GRID);
    }
    l.lds = table + (size_t)l.waves * each;
    // (the minima of the waves: 16 bytes each per count)
    if (l.lds < (size_t)l.waves * MK_COUNTS * 16) l.lds = (size_t)l.waves * MK_COUNTS * 16;
    return l;
}
