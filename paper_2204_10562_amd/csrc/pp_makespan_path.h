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
template <typename V> __device__ __forceinline__ V mk_times(V x, int k) {
    typedef typename mk_unsigned<V>::type U;
    return (V)((U)x * (U)(V)k);
}
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
#define MK_PICK_WAVES 4      // short lists of up to so many groups of 64: one workgroup schedules and picks

// LDS: PF and PB in pairs, then per wave one word per stage of each of its 64 plans, in rows an odd number
// of words apart: the device, and above it the stage's bound (0xffff: none such).
__host__ __device__ static inline size_t mk_path_table_bytes(int L) { return (size_t)(L + 1) * 16; }
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
    bool fits;        // no sum of the call leaves the integers V
    long long worst;  // the largest per-resource time (V = long long)
};

// The plan of xi stages in the wave's rows, of this lane (live: there is one).  PT: pairs (PF, PB).
template <int MODE, int NM, typename V>
__device__ __forceinline__ mk_plan_info mk_plan_path(const mk_args &a, const int *row, const long long *PT, int xi, bool live,
                                                     const int (&M)[NM], int limit, V (&T)[NM]) {
    constexpr bool narrow = sizeof(V) == 4;
    const int L = a.L, D = a.D, R = MODE == PP_SCHED_ADDITIVE ? xi : 2 * xi - 1;
    mk_path<V, NM> path;
    path.start();
    bool briefly[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) briefly[q] = MODE == PP_SCHED_DUPLEX || M[q] < 2 * R;
    struct piece { long long f[MK_AT_ONCE], b[MK_AT_ONCE]; };
    auto bound_of = [&](int w) { const int e = (unsigned)w >> 16; return e <= L ? e : L; };
    // transfer times into the stages n0 .. n0 + MK_AT_ONCE - 1 (before: the word of the stage before)
    auto ask = [&](piece &x, int n0, int before) {
#pragma unroll
        for (int u = 0; u < MK_AT_ONCE; ++u) {
            const int n = n0 + u;
            x.f[u] = x.b[u] = 0;
            if (n >= xi) continue;
            const int w = row[n], o = w & 0xffff, o0 = before & 0xffff, e0 = (unsigned)before >> 16;
            // (no branch around the loads: all of them are in flight together)
            const bool there = o < D && o0 < D && e0 >= 1 && e0 <= L && live;
            const size_t at = there ? (size_t)(unsigned)(o0 * D + o) * (unsigned)L + (unsigned)(e0 - 1) : 0;
            if (n) {
                x.f[u] = a.XF[at];
                x.b[u] = a.XB[at];
            }
            before = w;
        }
        return before;
    };
    piece now, then;
    int asked = ask(now, 0, 0), before = 0, e0 = 0;
    bool bad = false, torn = false;
    unsigned long long seen = 0;
    long long pf0 = PT[0], pb0 = PT[1], worst = 0;
    unsigned over = 0, most = 0;
    for (int n0 = 0; n0 < xi; n0 += MK_AT_ONCE) {
        if (n0 + MK_AT_ONCE < xi) asked = ask(then, n0 + MK_AT_ONCE, asked);
#pragma unroll
        for (int u = 0; u < MK_AT_ONCE; ++u) {
            const int n = n0 + u;
            if (n >= xi) continue;
            const int w = row[n], o = w & 0xffff, e = bound_of(w);
            bad |= o >= D;
            if (D <= 64) {
                bad |= (seen >> (o & 63)) & 1;
                seen |= 1ull << (o & 63);
            } else if (a.orderings) {
                for (int i = 0; i < n; ++i) bad |= (row[i] & 0xffff) == o;
            }
            torn |= (int)((unsigned)w >> 16) <= e0 || (int)((unsigned)w >> 16) > L;
            e0 = e;
            const long long pf = PT[2 * e], pb = PT[2 * e + 1];
            const long long F = pf - pf0, B = pb - pb0, cf = now.f[u], cb = now.b[u], s = F + B, x = cf + cb;
            pf0 = pf;
            pb0 = pb;
            if (narrow) {
                const long long all = MODE == PP_SCHED_ADDITIVE ? s + x : s | x;
                over |= (unsigned)(all >> 31);
                if (MODE == PP_SCHED_ADDITIVE) most = most > (unsigned)all ? most : (unsigned)all;
                else { most = most > (unsigned)s ? most : (unsigned)s; most = most > (unsigned)x ? most : (unsigned)x; }
            } else {
                worst = s > worst ? s : worst;
                worst = x > worst ? x : worst;
            }
            const bool last = n == xi - 1;
            if (MODE == PP_SCHED_ADDITIVE) {
                // the transfers over a stage's inbound link are part of its passes
                const V f = (V)(F + cf), b = (V)(B + cb);
                path.step(last ? mk_sum(f, b) : f, last ? (V)0 : b, 2 * (R - 1 - n), true, M, briefly);
            } else if (MODE == PP_SCHED_GPIPE) {
                path.step((V)cf, (V)cb, 0, false, M, briefly);
                path.step((V)F, (V)B, 0, false, M, briefly);
            } else {
                const int K = 2 * (R - 2 * n - 1);
                if (n) path.step((V)cf, (V)cb, K + 2, MODE != PP_SCHED_DUPLEX, M, briefly);
                path.step(last ? (V)s : (V)F, last ? (V)0 : (V)B, K, true, M, briefly);
            }
        }
        now = then;
    }
    torn |= e0 != L;
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        // (GPipe's order: two flow shops of M equal jobs, one after the other)
        if (MODE == PP_SCHED_GPIPE) T[q] = mk_sum(path.sum, mk_times(mk_sum(path.A, path.B), M[q] - 1));
        else T[q] = path.longest(q);
    }
    mk_plan_info i;
    // (a bad ordering is reported alone: its plan is not looked at)
    i.fault = !live ? 0 : bad ? PP_FAULT_ORDERING : torn ? PP_FAULT_BOUNDS : 0;
    i.worst = worst;
    i.fits = !narrow || !live || i.fault || (!over && (int)most <= limit);
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
// candidates, each wave some of the stage counts.
template <int MODE, int NM>
__device__ __forceinline__ void mk_path_body(const mk_args &a) {
    extern __shared__ __align__(16) int rows[];
    const int tid = threadIdx.x, lane = tid & 63, threads = blockDim.x, waves = threads >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S, L = a.L, D = a.D;
    long long *PT = (long long *)rows;
    for (int i = tid; i <= L; i += threads) {
        const long long f = a.PF[i], b = a.PB[i];
        PT[2 * i] = f;
        PT[2 * i + 1] = b;
    }
    int *mine = rows + mk_path_table_bytes(L) / 4 + wave * (mk_path_wave_bytes(S) / 4);
    int M[NM], mmax = 1;
    mk_counts<NM>(a, M);
#pragma unroll
    for (int q = 0; q < NM; ++q) mmax = M[q] > mmax ? M[q] : mmax;
    const bool listed = a.rlist && a.hdr->share_active;
    const long long todo = listed ? a.hdr->share_nreps : a.N, groups = (todo + 63) / 64;
    const int counts = a.search ? a.search : 1, per = a.search ? 1 : waves;
    tc_pair least[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) least[q] = {PP_INF64, INT64_MAX};
    __syncthreads();
    for (long long g = (long long)blockIdx.x * per + (a.search ? 0 : wave); g < groups; g += (long long)gridDim.x * per) {
        const long long at = g * 64 + lane;
        const bool live = at < todo;
        const long long c = !live ? 0 : listed ? pp_share_at(a.hdr, a.rlist, a.N, at) : at;
        const int held = (int)(todo - g * 64 < 64 ? todo - g * 64 : 64);  // plans of this group
        // (every other round of stage counts backwards: the waves' shares are alike)
        for (int turn = 0; turn * waves < counts || !a.search; ++turn) {
            const int k = turn * waves + (turn & 1 ? waves - 1 - wave : wave);
            const int xi = a.search ? k + 1 : S, SP = xi | 1;
            if (a.search && xi > counts) continue;
            const int bnd_off = a.search ? xi * (xi - 1) / 2 : a.bnd_off;
            const int limit = mk_split_limit(MODE == PP_SCHED_GPIPE ? 2ll * mmax + 4 * xi : mmax, xi);
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
                                      (int)((unsigned)(e[u] >= 1 && e[u] <= L ? e[u] : 0xffff) << 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int *row = mine + lane * SP;
            if (!a.orderings && live) {
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
            int T32[NM];
            mk_plan_info p = mk_plan_path<MODE, NM, int>(a, row, PT, xi, live, M, limit, T32);
#pragma unroll
            for (int q = 0; q < NM; ++q) T[q] = T32[q];
            if (__ballot(!p.fits)) {
                if (a.by_block) {
                    if (live) a.T_out[c * a.t_stride + a.t_off] = MK_NOT_TAKEN;
                    break;
                }
                p = mk_plan_path<MODE, NM, long long>(a, row, PT, xi, live, M, limit, T);
            }
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int slot = (int)blockIdx.y * NM + q;
                if (slot >= a.nM || !live) continue;
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

// The launch of mk_path_body: workgroups, waves in each, LDS, and whether the one workgroup picks the winners.
struct mk_path_launch { unsigned grid; int waves; size_t lds; int pick; };

static inline mk_path_launch mk_path_shape(const mk_args &a) {
    mk_path_launch l;
    const size_t table = mk_path_table_bytes(a.L), each = mk_path_wave_bytes(a.S);
    int most = (int)((64 * 1024 - table) / each);
    most = most < MK_PATH_WAVES ? most : MK_PATH_WAVES;
    const long long groups = (a.N + 63) / 64;
    l.pick = 0;
    if (a.search) {
        l.waves = a.search < most ? a.search : most;
        l.pick = a.part && groups == 1 && a.nM <= MK_COUNTS;
        l.grid = (unsigned)(groups < MK_PATH_GRID ? groups : MK_PATH_GRID);
    } else {
        // short lists: one workgroup that picks too; longer ones: a workgroup per compute unit first
        l.pick = a.part && groups <= most && groups <= MK_PICK_WAVES && a.nM <= MK_COUNTS;
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
