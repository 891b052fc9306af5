// Makespan (Eq. 2) of plans with replicated stages, S <= 16.
//
// T of Eq. 2 is the later of the last backward block on stage 0 and the ends of the AllReduces, which start when their
// stage's last backward pass has finished: the longest path of pp_makespan_path.h where it may also end at any stage's last
// backward item, with that stage's AllReduce behind it.  A walk that ends at stage q passes downwards from its
// last peak p to q only: in place of Sb(p) and B(p) stand the sum and the largest of the backward times from q to p,
// and down(p), or what is like it, is the largest over q (2 S - 1 peaks by up to S ends, three instructions each).
//
// What bounds it: instruction issue: about 100 instructions per stage for its times (quotients in doubles), as many
// for the minima over the links, and the walks.  40 320 orderings of 8 GPUs, plans of 1 .. 8 stages, M = 64: 134 -> 35 us
// (64-bit integer quotients and a sweep over all blocks per microbatch before); 3001 of 12 GPUs 58 -> 33 us.
#include <limits.h>

#include "pp_makespan_path.h"
#include "pp_prm.h"

// Waves of a workgroup, one per stage count where there are so many (8: 41 us for the 3001 orderings of 12 GPUs).
#define REP_WAVES 12

// LDS, in doubles: PF, PB, PA, the activation sizes, then a pair of bandwidths (there and back) per two devices, of
// 16 by 16, then the devices of 64 candidates and per wave a word (bound, replicas above it) per stage of their plans.
__host__ __device__ static inline size_t rep_table_bytes(int L) { return (size_t)5 * (L + 1) * 8 + 256 * 8; }
__host__ __device__ static inline size_t rep_rows_bytes(int D) { return (size_t)64 * (D | 1) * 4; }

__device__ __forceinline__ long long ceil_div64(long long x, long long y) { return x / y + (x % y != 0); }

struct rep_plan { long long T; int fault; bool fits; };

// The plan with S <= SMAX stages of this lane's candidate (work: there is one).  The cost model of Sec. III-B: stage s runs on
// k GPUs of consecutive ranks, a replica takes ceil(p / k) per microbatch, a transfer between stages of k' and
// k replicas ceil(d / (k' k min b)) with the minimum over the links between the two GPU sets, and a replicated stage
// ends with a ring AllReduce of ceil(2 (k-1) sum alpha / (k min b)) (Eq. 1).
// V = int: quotients below 2^30, of sizes below 2^53 held in doubles.  dev: the devices by rank, 4 bits each.
// (The stages in a loop, so that the code is fetched once: straight-line code for every S took as long for 3001 candidates as
// for 40 320.)
template <int SMAX, typename V>
__device__ __forceinline__ rep_plan rep_body(const mk_args &a, const double *tab, const int2 *links, const int *row,
                                             unsigned long long dev, bool work, bool bad, int S, int limit) {
    constexpr bool narrow = sizeof(V) == 4;
    constexpr V lowest = (V)((V)1 << (sizeof(V) * 8 - 2)) * -1;
    const int R = 2 * S - 1, L = a.L, L1 = L + 1, D = a.D, M = a.Ms[0];
    int fault = 0;
    {
        int prev = 0, used = 0;
        for (int s = 0; s < S; ++s) {
            const int e = row[s] & 0xffff, k = (int)((unsigned)row[s] >> 16);
            if (e <= prev || e > L || k < 1 || k > D) fault = PP_FAULT_BOUNDS;
            prev = e;
            used += k;
        }
        if (prev != L || used != D) fault = PP_FAULT_BOUNDS;
        if (bad) fault |= PP_FAULT_ORDERING;
    }
    const bool ok = work && !fault;
    // the walks: sums and largest times so far, and per end what comes on top of the sum of all backward times so far
    // (ends still to come: less than anything) and the largest of them since
    V sa = 0, sb = 0, A = 0, brief = 0, at = lowest * 2, up = at, down = at, both = at, tail[SMAX], most[SMAX];
#pragma unroll
    for (int q = 0; q < SMAX; ++q) { tail[q] = lowest; most[q] = 0; }
    auto step = [&](V x, V y, int K) {
        const V before = mk_sum(sa, sb);
        sa = mk_sum(sa, x);
        sb = mk_sum(sb, y);
        A = mk_larger(A, x);
        // the last part of a walk with k sweeps to spend on the way down
        auto ending = [&](int k) {
            V v = lowest;
#pragma unroll
            for (int q = 0; q < SMAX; ++q) v = mk_larger(v, mk_sum(tail[q], mk_times(most[q], k)));
            return mk_sum(mk_sum(sa, sb), v);
        };
#pragma unroll
        for (int q = 0; q < SMAX; ++q) most[q] = mk_larger(most[q], y);
        const V d = ending(K);
        if (M - 2 >= K) {
            const V c = mk_sum(x, y), u = mk_sum(mk_sum(sa, sb), mk_times(A, K));
            at = mk_larger(at, mk_less(mk_times(c, M - 2 - K), before));
            up = mk_larger(up, mk_sum(at, u));
            down = mk_larger(down, mk_sum(at, d));
            both = mk_larger(both, mk_larger(mk_sum(up, d), mk_sum(down, u)));
        }
        if (M < 2 * R) {
            const int m = M - 1, k = K < m ? K : m;
            const V w = mk_sum(ending(m), mk_times(A, k)), z = mk_sum(k == K ? d : ending(k), mk_times(A, m));
            brief = mk_larger(brief, mk_larger(w, z));
        }
    };
    long long worst = 0, amax = 0;
    double largest = 0.0;  // of the quotients
    int e0 = 0, n = 0, k0 = 0;
    auto quotient = [&](double x, double den, double inv) {
        const double q = __builtin_trunc(x * inv), rem = __builtin_fma(-q, den, x);
        largest = q > largest ? q : largest;
        return (int)q + (rem > 0.0) + (rem > den);
    };
    for (int s = 0; s < S; ++s) {
        const int e = ok ? row[s] & 0xffff : 0, k = ok ? (int)((unsigned)row[s] >> 16) : 0;
        // the links inside the stage, and those from the stage before and back
        int m = INT_MAX, mf = INT_MAX, mb = INT_MAX;
        long long wm = PP_INF64, wf = PP_INF64, wb = PP_INF64;
        for (int v = n; v < n + k; ++v) {
            const int dv = (int)(dev >> (4 * v)) & 15;
            if (narrow) {
                // (four reads in flight; beyond v a link once more)
                for (int u0 = n - k0; u0 < v; u0 += 4) {
                    int2 x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int u = u0 + j < v ? u0 + j : u0;
                        x[j] = links[((int)(dev >> (4 * u)) & 15) * 16 + dv];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool inside = (u0 + j < v ? u0 + j : u0) >= n;
                        const int least = x[j].x < x[j].y ? x[j].x : x[j].y;
                        m = inside && least < m ? least : m;
                        mf = !inside && x[j].x < mf ? x[j].x : mf;
                        mb = !inside && x[j].y < mb ? x[j].y : mb;
                    }
                }
            } else {
                for (int u = n - k0; u < v; ++u) {
                    const int du = (int)(dev >> (4 * u)) & 15;
                    const bool inside = u >= n;
                    const long long x = a.bw[du * D + dv], y = a.bw[dv * D + du], least = x < y ? x : y;
                    wm = inside && least < wm ? least : wm;
                    wf = !inside && x < wf ? x : wf;
                    wb = !inside && y < wb ? y : wb;
                }
            }
        }
        V F = 0, B = 0, cf = 0, cb = 0, As = 0;
        if (narrow) {
            const double kd = ok ? (double)k : 1.0, inv = prm_inv(kd);
            F = quotient(tab[e] - tab[e0], kd, inv);
            B = quotient(tab[L1 + e] - tab[L1 + e0], kd, inv);
            if (__ballot(k > 1)) {
                const double den = kd * (double)m;
                const int r = quotient(k > 1 ? 2.0 * (kd - 1.0) * (tab[2 * L1 + e] - tab[2 * L1 + e0]) : 0.0, den, prm_inv(den));
                As = k > 1 ? r : 0;
            }
            if (s) {
                const double kk = ok ? kd * (double)k0 : 1.0, df = kk * (double)mf, db = kk * (double)mb;
                cf = quotient(tab[3 * L1 + e0], df, prm_inv(df));
                cb = quotient(tab[4 * L1 + e0], db, prm_inv(db));
            }
        } else if (ok) {
            F = (V)ceil_div64(a.PF[e] - a.PF[e0], k);
            B = (V)ceil_div64(a.PB[e] - a.PB[e0], k);
            if (k > 1) As = (V)ceil_div64(2 * (long long)(k - 1) * (a.PA[e] - a.PA[e0]), (long long)k * wm);
            if (s) {
                cf = (V)ceil_div64(a.actf[e0 - 1], (long long)k0 * k * wf);
                cb = (V)ceil_div64(a.actb[e0 - 1], (long long)k0 * k * wb);
            }
        }
        const V w = mk_larger(mk_sum(F, B), mk_sum(cf, cb));
        worst = w > worst ? w : worst;
        amax = As > amax ? As : amax;
        e0 = e;
        n += k;
        k0 = k;
        const int K = 2 * (R - 2 * s - 1);
        if (s) step(cf, cb, K + 2);
        // (this stage is an end from its own peak on)
#pragma unroll
        for (int q = 0; q < SMAX; ++q)
            if (q == s) { tail[q] = mk_less(As, sb); most[q] = 0; }
        step(s == S - 1 ? mk_sum(F, B) : F, s == S - 1 ? (V)0 : B, K);
    }
    if (ok && !narrow) {
        fault |= overflow_fault(worst, M, S);
        if (amax >= PP_CAP62 / 2) fault |= PP_FAULT_OVERFLOW;
    }
    rep_plan out;
    out.fault = work ? fault : 0;
    out.T = mk_larger(both, brief);
    out.fits = !narrow || !ok || (largest < (double)PP_TIME_CAP && worst <= limit);
    return out;
}

// Workgroups take 64 candidates, their waves some of the stage counts each.
template <int SMAX>
__global__ __launch_bounds__(64 * REP_WAVES) void k_rep_makespan(mk_args a) {
    extern __shared__ __align__(16) double rep_lds[];
    const int tid = threadIdx.x, lane = tid & 63, T = blockDim.x, waves = T >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = a.L, L1 = L + 1, D = a.D, DP = D | 1;
    double *tab = rep_lds;
    int2 *links = (int2 *)(tab + 5 * L1);
    int *so = (int *)(links + 256), *mine = so + 64 * DP + wave * 64 * DP;
    // sizes that doubles and ints hold: all of the launch sees the same
    bool exact = a.PA[L] < (1ll << 53) / (2 * D) && a.PF[L] < 1ll << 53 && a.PB[L] < 1ll << 53;
    for (int l = tid; l <= L; l += T) {
        const long long f = l ? a.actf[l - 1] : 0, b = l ? a.actb[l - 1] : 0;
        tab[l] = (double)a.PF[l];
        tab[L1 + l] = (double)a.PB[l];
        tab[2 * L1 + l] = (double)a.PA[l];
        tab[3 * L1 + l] = (double)f;
        tab[4 * L1 + l] = (double)b;
        exact &= l == L || (f >= 0 && b >= 0 && f < 1ll << 53 && b < 1ll << 53);  // (the last entry is ignored)
    }
    for (int t = tid; t < D * D; t += T) {
        const int u = t / D, v = t - u * D;
        const long long x = a.bw[t], y = a.bw[v * D + u];
        links[u * 16 + v] = make_int2((int)x, (int)y);
        exact &= u == v || (x > 0 && x < 1ll << 30);
    }
    exact = __syncthreads_and(exact);
    tc_pair least[1] = {{PP_INF64, INT64_MAX}};
    const long long groups = (a.N + 63) / 64;
    for (long long g = blockIdx.x; g < groups; g += gridDim.x) {
        const long long c0 = g * 64, c = c0 + lane;
        const bool live = c < a.N;
        __syncthreads();
        for (int t = tid; t < 64 * D; t += T) {
            const int i = t / D, n = t - i * D;
            so[i * DP + n] = c0 + i < a.N ? a.orderings[c0 * D + t] : 0;
        }
        __syncthreads();
        unsigned long long dev = 0;
        unsigned seen = 0;
        bool bad = false;
        for (int n = 0; n < D; ++n) {
            const int d = so[lane * DP + n];
            bad |= d < 0 || d >= D || (seen >> (d & 15) & 1);
            seen |= 1u << (d & 15);
            dev |= (unsigned long long)(d & 15) << (4 * n);
        }
        for (int turn = 0; turn * waves < D; ++turn) {
            // (every other round backwards: the waves' shares are alike)
            const int xi = turn * waves + (turn & 1 ? waves - 1 - wave : wave) + 1;
            if (xi > D) continue;
            const long long tri = a.bnd_stride;
            const int at = xi * (xi - 1) / 2;
            __builtin_amdgcn_wave_barrier();
            for (int t0 = lane; t0 < 64 * xi; t0 += 64 * 4) {
                int e[4], k[4], to[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int t = t0 + 64 * u, i = t / xi, n = t - i * xi;
                    to[u] = t < 64 * xi && c0 + i < a.N ? i * DP + n : -1;
                    e[u] = to[u] >= 0 ? a.bounds[(c0 + i) * tri + at + n] : 0;
                    k[u] = to[u] >= 0 ? a.reps[(c0 + i) * tri + at + n] : 0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (to[u] >= 0) mine[to[u]] = (e[u] >= 0 && e[u] <= L ? e[u] : 0) | (k[u] >= 0 && k[u] <= D ? k[u] : 0) << 16;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const bool none = live && a.W[c * D + xi - 1] == PP_INF64;  // no plan with so many stages
            rep_plan p = {};
            const int limit = exact ? pp_time_limit(a.Ms[0], xi) : -1;
            if (limit >= 0) p = rep_body<SMAX, int>(a, tab, links, mine + lane * DP, dev, live && !none, bad, xi, limit);
            if (limit < 0 || __ballot(!p.fits))
                p = rep_body<SMAX, long long>(a, tab, links, mine + lane * DP, dev, live && !none, bad, xi, limit);
            if (live) {
                if (p.fault) pp_raise(a.status, p.fault);
                const long long t = none || p.fault ? PP_INF64 : p.T;
                a.T_out[c * D + xi - 1] = t;
                least[0] = tc_min(least[0], {t, c * D + xi - 1});
            }
        }
    }
    mk_leave_least<1>(a, least, (tc_pair *)rep_lds);
}

int mk_launch_replicated(const mk_args &a, hipStream_t st, long long *n_part) {
    const long long groups = (a.N + 63) / 64;
    const unsigned grid = (unsigned)(groups < MK_PATH_GRID ? groups : MK_PATH_GRID);
    mk_args b = a;
    b.pick_here = grid == 1;
    *n_part = b.pick_here ? 0 : grid;
    const size_t fixed = rep_table_bytes(a.L) + rep_rows_bytes(a.D);
    int waves = a.D < REP_WAVES ? a.D : REP_WAVES;
    while (waves > 1 && fixed + waves * rep_rows_bytes(a.D) > 64 * 1024) --waves;
    const size_t lds = fixed + waves * rep_rows_bytes(a.D);
    const dim3 block(64 * waves);
    if (a.D <= 4) hipLaunchKernelGGL(k_rep_makespan<4>, dim3(grid), block, lds, st, b);
    else if (a.D <= 8) hipLaunchKernelGGL(k_rep_makespan<8>, dim3(grid), block, lds, st, b);
    else if (a.D <= 12) hipLaunchKernelGGL(k_rep_makespan<12>, dim3(grid), block, lds, st, b);
    else hipLaunchKernelGGL(k_rep_makespan<16>, dim3(grid), block, lds, st, b);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
