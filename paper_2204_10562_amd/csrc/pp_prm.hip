// Partition, replication and mapping (PRM, Alg. 4; recursion for W(l, xi, r, i) in Sec. IV-B)
// for a batch of device orderings: the dynamic program over (layers, stages, replicas of the
// last stage, GPUs used) with the AllReduce term of Eq. 1, for every stage count at once.
//
//   W(l, xi, r, i) = min over l' in [xi-1, l-1], r' in [1, i-r] of
//                    max{ W(l', xi-1, r', i-r),  M (c^f + c^b),  M (F + B) + A }
//   W(l, 1, i, i)  = M (F + B) + A of layers [0, l) on all i GPUs
// where, for the last stage = layers [l', l) on the r GPUs of ranks [i-r, i):
//   F = ceil(sum p^f / r), B = ceil(sum p^b / r)            (per-replica times, Sec. III-B)
//   A = ceil(2 (r-1) sum alpha / (r min b)), 0 for r = 1    (Eq. 1; min over the replica set)
//   c^f = ceil(d^f / (r' r min b_{v',v})), c^b = ceil(d^b / (r' r min b_{v,v'}))
//         (v' in the r' GPUs of ranks [i-r-r', i-r), v in the last stage's).
// The listing scans l' ascending, then r' ascending, and replaces its best only on strict
// improvement: the minimiser kept is the first in (l', r') order.
//
// Where the cells that a good plan can use are few, k_prm_band (pp_prm_band.hip) has planned the launch when this
// kernel starts; it does the others.
//
// One workgroup of two waves per candidate (persistent over candidates), one lane per cell l.  State
// (xi, r, i) depends only on states with fewer GPUs, so states are visited by ascending i, and with
// int32 values each wave does half of the states of an i on its own, without barriers.
// All states with the same (r, i) share the last stage's terms, which are made division-free:
// with Q[l] = floor(P[l] / r), R[l] = P[l] mod r,  ceil((P[l] - P[l']) / r) =
// Q[l] - Q[l'] + (R[l] > R[l']); so the stage term is U[l] - U[l'] + (remainder compares) with
// U = M (QF + QB) + QA; the channel term X[r'][l'] = M (c^f + c^b) is computed once per (r, i)
// too.  Neither the sub-problem nor the channel term depends on l, and the last stage's term
// does not depend on r'; max with the latter commutes with the minimum over r', so per state
//   Gmin[l'] = min over r' of max(W(l', xi-1, r', i-r), X[r'][l'])
// is built once in LDS and a cell is
//   W(l, xi, r, i) = min over l' of max(Gmin[l'], last stage [l', l)).
// The last stage's term falls as l' grows, so with int32 values the cell is found by a binary
// search (see the cells); int64 values pass over l' from l - 1 down with an early exit.  The r'
// that goes with the chosen l' is the first one whose value reaches the minimum; with int32
// values it is worked out for the plans' cells only.
// States that use all D GPUs are needed at l = L only: the lanes share the scan of l'.
//
// Bound by vector instructions and the latency of the short phases of a state.  L = 128, D = 8, all
// 40320 orderings, whole call: 9.40 ms with a pass over l' per cell and 64-bit divisions, 8.37 ms with
// the divisions in doubles, 5.11 ms with the search (82 K, 70 K and 33 K vector instructions per
// candidate), 3.95 ms with a wave per state instead of a workgroup per state and three barriers in
// it (L = 8, where one wave was idle: 3.2 -> 2.2 ms).
#include "pp_common.h"
#include "pp_dp_row.h"
#include "pp_prm.h"

#define PRM_THREADS 128
// Fewest layers for which a cell's split is searched rather than scanned for (int32 values).  All
// 40320 orderings of 8 GPUs, whole call, scan / search in ms: 2.60 / 2.65 at L = 32, 2.80 / 2.73 at
// 48, 2.99 / 2.87 at 64, 4.29 / 3.68 at 72 (a second chunk of positions), 4.82 / 3.85 at 112.
#define PRM_SEARCH_MIN_L 40

// Bytes of per-workgroup scratch: W and the minimising (l', r') of every state and cell, and
// the minima of the bandwidth matrix over rank sets.
static inline size_t prm_slot_bytes(int L, int D) {
    size_t cells = (size_t)prm_states(D) * (L + 1);
    size_t minima = (size_t)(D + 1) * (D + 1) * (D + 1) * 2 + (size_t)(D + 1) * (D + 1);
    return pp_align256(cells * 8) + pp_align256(cells * 4) + pp_align256(minima * 8);
}

static inline size_t prm_lds_bytes(int L, int D) {
    // PF, PB, PA (int64), one row record per layer position (32 bytes in the int64 form),
    // X (int64, D-1 rows)
    // (the three prefix arrays are padded to an even length so that the records are 16-byte aligned)
    return (size_t)(L + 2) * (3 * 8) + (size_t)(L + 1) * 32 + (size_t)(D > 1 ? D - 1 : 1) * (L + 1) * 8 + 64;
}

// The int32 form: two sets of records (16 bytes) and channel terms (one row less in the second), and of
// Gmin where cells are searched for.  Without those it is less than the above.
static inline size_t prm_search_lds_bytes(int L, int D) {
    return (size_t)(L + 2) * (3 * 8) + (size_t)(L + 1) * (2 * 16 + (2 * D - 1) * 4);
}

struct prm_key {
    long long v;
    int lp, rp;
};

__device__ __forceinline__ bool prm_less(const prm_key &a, const prm_key &b) {
    if (a.v != b.v) return a.v < b.v;
    if (a.lp != b.lp) return a.lp < b.lp;
    return a.rp < b.rp;
}

// Values are int64, or int32 when every finite value of the launch is known to stay below
// 2^30 (decided on the device from bounds on the stage and channel terms) and every size below
// 2^53, so that quotients can be had by double arithmetic.
template <bool WIDE> struct prm_val { using V = int; };
template <> struct prm_val<true> { using V = long long; };

// What the cell loop reads per layer position l' (one LDS access in the int32 form):
//   g  = Gmin[l'] of the current state
//   u  = U[l'], ra = remainder of the AllReduce quotient   (current (r, i))
//   oh = (1 << RF[l']) | (1 << (16 + RB[l'])), the remainders of the two compute quotients as
//        one-hot bits, so that [RF[l] > RF[l']] + [RB[l] > RB[l']] is the popcount of oh
//        masked with ((1 << RF[l]) - 1) | (((1 << RB[l]) - 1) << 16).
template <bool WIDE> struct alignas(16) prm_row { int g, u, ra, oh; };
template <> struct alignas(16) prm_row<true> { long long g, u, ra; int oh, pad; };

struct prm_shared {
    int o[16];
    int fault, keep, wide;
    unsigned long long amax_f, amax_b, bmin, bmax;
    prm_key red[PRM_THREADS / 64];
};

template <bool WIDE>
__device__ void prm_run(const prm_args &a, unsigned char *smem, prm_shared &sh) {
    using V = typename prm_val<WIDE>::V;
    using Row = prm_row<WIDE>;
    const V INF = WIDE ? (V)PP_INF64 : (V)PP_INF32;
    const int L = a.L, D = a.D, tid = threadIdx.x, B = blockDim.x;
    const long long M = a.M;
    const V Mv = (V)a.M;
    const int L1 = L + 1, D1 = D + 1;
    const int L1p = (L1 + 1) & ~1;  // even, so that what follows the int64 arrays is 16-byte aligned
    long long *PF = (long long *)smem, *PB = PF + L1p, *PA = PB + L1p;
    // int32 values: every wave does states of its own (see the states), with its own records, channel
    // terms and minima (WV); int64 values: the workgroup does one state at a time
    constexpr int WV = WIDE ? 1 : 2;
    const int lane = tid & 63, wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tl = WIDE ? tid : lane, BL = WIDE ? B : 64, part = WIDE ? 0 : wib;
    Row *Q = (Row *)(PA + L1p) + (size_t)part * L1;                                     // [L1]
    V *X = (V *)((Row *)(PA + L1p) + (size_t)WV * L1) + (size_t)part * (D - 1) * L1;    // [D-1][L1] (part 1: [D-2])
    // int32 values, cells searched for: Gmin; the g field of a record then holds H(l' + 1) (see the cells)
    int *Gr = (int *)((Row *)(PA + L1p) + (size_t)WV * L1) + (size_t)(2 * D - 3 + part) * L1;
    const int NS = prm_states(D), tri = D * (D + 1) / 2;
    char *slot = a.scratch + (size_t)blockIdx.x * a.slot_bytes;
    V *Wt = (V *)slot;                                                   // [NS][L1]
    unsigned *At = (unsigned *)(slot + pp_align256((size_t)NS * L1 * 8));  // l' | r' << 16
    long long *bfwd = (long long *)((char *)At + pp_align256((size_t)NS * L1 * 4));  // [p][rp][r]
    long long *bbwd = bfwd + (size_t)D1 * D1 * D1;
    long long *bin = bbwd + (size_t)D1 * D1 * D1;                        // [n][r]
    // int32 values: the minima are kept as the denominators they end up in (doubles in the same
    // places); the arrays of prefix sums in LDS hold the activation sizes at the cuts and the prefix
    // sums of the parameter sizes as doubles; and what the last stage's compute terms are at every
    // position (M (QF + QB), one-hot remainders) is tabled per number of replicas behind the table of
    // W, which leaves half of its area.  (D >= 2.)
    double *dfwd = (double *)bfwd, *dbwd = (double *)bbwd, *din = (double *)bin;
    double *AF = (double *)PF, *AB = (double *)PB, *PAd = (double *)PA;
    int2 *UT = (int2 *)(slot + (((size_t)NS * L1 * 4 + 7) & ~(size_t)7));  // [r - 1][L1]
    if constexpr (!WIDE) {
        for (int r = 1; r <= D; ++r)
            for (int l = tid; l <= L; l += B) {
                const long long qf = PF[l] / r, qb = PB[l] / r;
                UT[(size_t)(r - 1) * L1 + l] = make_int2((int)(M * (qf + qb)), (1 << (int)(PF[l] - qf * r)) | (1 << (16 + (int)(PB[l] - qb * r))));
            }
        __syncthreads();
        for (int l = tid; l <= L; l += B) {
            AF[l] = l >= 1 && l < L ? (double)a.actf[l - 1] : 0.0;
            AB[l] = l >= 1 && l < L ? (double)a.actb[l - 1] : 0.0;
            PAd[l] = (double)PA[l];
        }
        if (lane == 0) { Q[0].u = 0; Q[0].ra = 0; Q[0].oh = 0x10001; }
        __syncthreads();
    }
    auto sync = [&]() {
        if constexpr (WIDE) __syncthreads();
        else row_lds_sync();
    };
    const bool search = !WIDE && L >= PRM_SEARCH_MIN_L && a.search;

    // A workgroup walks a contiguous chunk of candidates.  State (xi, r, i) depends only on the
    // first i devices of the ordering, so whatever the previous candidate shares as a prefix is
    // kept (with all D! orderings in lexicographic order most of the table is).
    const long long chunk = (a.N + gridDim.x - 1) / gridDim.x;
    const long long c_first = (long long)blockIdx.x * chunk;
    const long long c_end = c_first + chunk < a.N ? c_first + chunk : a.N;
    bool have_prev = false;
    for (long long c = c_first; c < c_end; ++c) {
        __syncthreads();
        // ---- ordering
        if (tid == 0) {
            int bad = 0, same = 0;
            bool eq = have_prev;
            for (int n = 0; n < D; ++n) {
                int d = a.ord[c * D + n];
                if (d < 0 || d >= D) bad = 1;
                for (int q = 0; q < n; ++q) bad |= (sh.o[q] == d);
                eq = eq && sh.o[n] == d;
                same += eq;
                sh.o[n] = d;
            }
            sh.fault = bad;
            sh.keep = same < D ? same : D - 1;  // the states on all D GPUs are always redone
        }
        __syncthreads();
        const int keep = sh.keep;
        have_prev = !sh.fault;
        if (sh.fault) {
            if (tid == 0) pp_raise(a.status, PP_FAULT_ORDERING);
            for (int n = tid; n < D; n += B) a.W_out[c * D + n] = PP_INF64;
            for (int n = tid; n < tri; n += B) { a.bounds_out[c * tri + n] = 0; a.reps_out[c * tri + n] = 0; }
            continue;
        }
        const int *o = sh.o;
        // ---- minima of the bandwidth matrix over rank sets
        // bfwd[p][rp][r]: links from ranks [p-rp, p) to ranks [p, p+r); bbwd: the other direction
        for (int t = tid; t < D1 * D1 * D1; t += B) {
            const int p = t / (D1 * D1), rp = (t / D1) % D1, r = t % D1;
            if (p < 1 || rp < 1 || r < 1 || rp > p || p + r > D || p + r <= keep) continue;
            long long mf = PP_INF64, mb = PP_INF64;
            for (int u = p - rp; u < p; ++u)
                for (int v = p; v < p + r; ++v) {
                    long long x = a.bw[(size_t)o[u] * D + o[v]], y = a.bw[(size_t)o[v] * D + o[u]];
                    mf = x < mf ? x : mf;
                    mb = y < mb ? y : mb;
                }
            if constexpr (WIDE) {
                bfwd[t] = mf;
                bbwd[t] = mb;
            } else {
                dfwd[t] = (double)(rp * r) * (double)mf;
                dbwd[t] = (double)(rp * r) * (double)mb;
            }
        }
        // bin[n][r]: ordered pairs inside ranks [n-r, n)
        for (int t = tid; t < D1 * D1; t += B) {
            const int n = t / D1, r = t % D1;
            if (n < 1 || r < 2 || r > n || n <= keep) continue;
            long long m = PP_INF64;
            for (int u = n - r; u < n; ++u)
                for (int v = n - r; v < n; ++v)
                    if (u != v) {
                        long long x = a.bw[(size_t)o[u] * D + o[v]];
                        m = x < m ? x : m;
                    }
            if constexpr (WIDE) bin[t] = m;
            else din[t] = (double)r * (double)m;
        }
        __syncthreads();

        // ---- states by ascending number of GPUs
        for (int i = keep + 1; i <= D; ++i) {
            const bool top = i == D;  // all GPUs in use: only cell L is needed
            for (int r = 1; r <= i; ++r) {
                // r = 1, 4, 5, 8, .. by wave 0 and 2, 3, 6, 7, .. by wave 1: about as many states each
                if (!WIDE && ((r >> 1) & 1) != part) continue;
                // Last stage on r replicas, ranks [i-r, i): division-free form of its terms, and
                // the channel term X[r'][l'] = M (c^f + c^b) towards r' replicas on ranks
                // [i-r-r', i-r); both are shared by every stage count.
                const int n0 = i - r;  // GPUs of the sub-problem
                if constexpr (WIDE) {
                    const long long den = r > 1 ? (long long)r * bin[i * D1 + r] : 1;
                    for (int l = tl; l <= L; l += BL) {
                        long long qf = PF[l] / r, qb = PB[l] / r;
                        long long num = 2 * (long long)(r - 1) * PA[l];
                        long long qa = num / den;
                        Q[l].u = (V)(M * (qf + qb) + qa);
                        Q[l].ra = (V)(num - qa * den);
                        Q[l].oh = (1 << (int)(PF[l] - qf * r)) | (1 << (16 + (int)(PB[l] - qb * r)));
                    }
                    for (int t = tl; t < n0 * L1; t += BL) {
                        const int rp = 1 + t / L1, lp = t % L1;
                        V x = INF;
                        if (lp >= 1 && lp <= L - 1) {
                            const size_t at = ((size_t)n0 * D1 + rp) * D1 + r;
                            x = (V)(M * (cdiv64(a.actf[lp - 1], (long long)rp * r * bfwd[at]) +
                                         cdiv64(a.actb[lp - 1], (long long)rp * r * bbwd[at])));
                        }
                        X[(size_t)(rp - 1) * L1 + lp] = x;
                    }
                } else {
                    const double den = r > 1 ? din[i * D1 + r] : 1.0, inv = prm_inv(den), times = 2.0 * (r - 1);
                    const int2 *ut = UT + (size_t)(r - 1) * L1;
                    for (int l = tl + 1; l <= L; l += BL) {
                        const int2 u = ut[l];
                        int ra = 0;
                        const int qa = r > 1 ? prm_floor_div(times * PAd[l], den, inv, ra) : 0;
                        Q[l].u = u.x + qa;
                        Q[l].ra = ra;
                        Q[l].oh = u.y;
                    }
                    for (int rp = 1; rp <= n0; ++rp) {
                        const size_t at = ((size_t)n0 * D1 + rp) * D1 + r;
                        const double f = dfwd[at], b = dbwd[at], finv = prm_inv(f), binv = prm_inv(b);
                        V *Xr = X + (size_t)(rp - 1) * L1;
                        for (int lp = tl; lp < L; lp += BL)
                            Xr[lp] = (int)M * (prm_ceil_div(AF[lp], f, finv) + prm_ceil_div(AB[lp], b, binv));
                    }
                }
                sync();
                // the last stage [l', l): M (F + B) + A, from the records of l' and l
                auto last_stage = [&](const Row &q, const Row &ql, int mask) -> V {
                    const int flags = __popc((unsigned)(q.oh & mask));  // 0, 1 or 2
                    const V extra = WIDE ? Mv * (V)flags : (V)__mul24(flags, (int)Mv);  // M < 2^20 here
                    return ql.u - q.u + extra + (V)(ql.ra > q.ra);
                };
                auto mask_of = [](int oh) -> int {
                    // remainders (f, b) one-hot at bits f and 16 + b -> all lower bits of each half
                    return oh - 0x10001;
                };
                for (int xi = 1; xi <= i - r + 1; ++xi) {
                    const int sid = prm_sid(i, xi, r);
                    V *Ws = Wt + (size_t)sid * L1;
                    unsigned *As = At + (size_t)sid * L1;
                    if (xi == 1) {
                        // a single stage must take all i GPUs
                        for (int l = top ? L + tl : tl + 1; l <= L; l += BL) {
                            Ws[l] = (r == i) ? last_stage(Q[0], Q[l], mask_of(Q[l].oh)) : INF;
                            As[l] = 0;
                        }
                        continue;  // touches no LDS array that the next state rewrites
                    }
                    const int nrp = n0 - (xi - 2);  // r' = 1..nrp leave >= 1 GPU per earlier stage
                    // Gmin[l'] = min over r' of max(W(l', xi-1, r', n0), X[r'][l']).  The last
                    // stage's term does not depend on r', and max with it commutes with this min.
                    for (int lp = tl; lp < L; lp += BL) {
                        V g = INF;
                        if (lp >= xi - 1) {
                            // four loads in flight at a time; a clamped r' repeats the last one
                            const V *Wsub = Wt + (size_t)prm_sid(n0, xi - 1, 1) * L1 + lp;  // r' = 1, 2, ...
                            for (int rp0 = 1; rp0 <= nrp; rp0 += 4) {
                                V w[4], x[4];
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const int rp = rp0 + k <= nrp ? rp0 + k : nrp;
                                    w[k] = Wsub[(size_t)(rp - 1) * L1];
                                    x[k] = X[(size_t)(rp - 1) * L1 + lp];
                                }
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const V m = w[k] > x[k] ? w[k] : x[k];
                                    g = m < g ? m : g;
                                }
                            }
                        }
                        if (search) Gr[lp] = (int)g;
                        else Q[lp].g = g;
                    }
                    sync();
                    // first r' (ascending) whose value reaches the minimum v found at l'
                    auto first_rp = [&](int lp, int l, V v) -> int {
                        const V last = last_stage(Q[lp], Q[l], mask_of(Q[l].oh));
                        for (int rp = 1; rp <= nrp; ++rp) {
                            V w = Wt[(size_t)prm_sid(n0, xi - 1, rp) * L1 + lp];
                            V x = X[(size_t)(rp - 1) * L1 + lp];
                            w = w > x ? w : x;
                            if ((w > last ? w : last) == v) return rp;
                        }
                        return 0;
                    };
                    if (!top && search) {
                        // The minimum over l' of max(G[l'], last stage [l', l)) by a search, as in
                        // pp_dp_row.h: G = Gmin, and the last stage's term falls as l' grows.  With
                        // H(j) = min_{k>=j} G[k] over the whole row, split j is done for iff its last
                        // stage exceeds H(j + 1); the first that is not is the crossing.  Here the last
                        // stage's term can be equal at neighbouring splits (quotients): the lowest of
                        // those with G no larger is taken.
                        int carry = PP_INF32;
                        for (int c = L & ~63; c >= 0; c -= 64) {
                            const int lp = c + lane;
                            const int m = row_suffix_min(lp >= xi - 1 && lp < L ? Gr[lp] : PP_INF32, carry, lane);
                            carry = __builtin_amdgcn_readlane(m, 0);
                            if (lp >= 1 && lp <= L) Q[lp - 1].g = m;
                        }
                        sync();
                        const int lo = xi - 1;
                        int steps = 1;
                        while ((1 << steps) - 1 < L / xi + L / (8 * xi) + 3) ++steps;
                        for (int l = tl + 1; l <= L; l += BL) {
                            const Row ql = Q[l];
                            const int mask = mask_of(ql.oh);
                            int pos = l - 1;
                            for (;;) {
                                const int from = pos;
                                for (int st = 1 << (steps - 1); st; st >>= 1) {
                                    const int k = row_imax(pos - st, lo);
                                    const Row q = Q[k];
                                    pos = k < pos && last_stage(q, ql, mask) <= q.g ? k : pos;
                                }
                                if (!__ballot(pos > lo && pos == from - ((1 << steps) - 1))) break;
                            }
                            V best = INF;
                            int blp = 0;
                            if (l > lo) {
                                const Row q = Q[pos];
                                const V last = last_stage(q, ql, mask), g = Gr[pos];
                                if (g <= q.g) {
                                    best = g > last ? g : last;
                                    blp = pos;
                                    for (int k = pos - 1; k >= lo && best != INF && last_stage(Q[k], ql, mask) <= best; --k)
                                        blp = Gr[k] <= best ? k : blp;
                                } else {
                                    int e = pos + 1;
                                    while (e < l && Gr[e] > q.g) ++e;
                                    if (e < l) {
                                        best = q.g;
                                        blp = e;
                                    } else {
                                        for (int k = l - 1; k >= lo; --k) {
                                            const V lk = last_stage(Q[k], ql, mask), gk = Gr[k];
                                            if (lk > best) break;
                                            const V t = gk > lk ? gk : lk;
                                            if (t <= best) { best = t; blp = k; }
                                        }
                                    }
                                }
                            }
                            // (which r' goes with it is worked out for the plans only)
                            Ws[l] = best;
                            As[l] = (unsigned)blp;
                        }
                    } else if (!top) {
                        for (int l = tl + 1; l <= L; l += BL) {
                            const Row ql = Q[l];
                            const int mask = mask_of(ql.oh);
                            V best = INF;
                            int blp = 0;
                            // Splits from l-1 downwards: the last stage's term grows as l'
                            // falls, so once it alone exceeds the best value no lower l' can
                            // match it.  '<=' keeps the lowest l' among equal values, which is
                            // what the ascending scan with '<' of the listing keeps.
                            int lp = l - 1;
                            for (; lp - 3 >= xi - 1; lp -= 4) {
                                Row q[4];
#pragma unroll
                                for (int k = 0; k < 4; ++k) q[k] = Q[lp - k];
                                V last = 0;
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    last = last_stage(q[k], ql, mask);
                                    const V t = q[k].g > last ? q[k].g : last;
                                    if (t <= best) { best = t; blp = lp - k; }
                                }
                                if (last > best) { lp = xi - 2; break; }  // nothing below can win
                            }
                            for (; lp >= xi - 1; --lp) {
                                const Row q = Q[lp];
                                const V last = last_stage(q, ql, mask);
                                if (last > best) break;
                                const V t = q.g > last ? q.g : last;
                                if (t <= best) { best = t; blp = lp; }
                            }
                            Ws[l] = best;
                            As[l] = (unsigned)blp;
                            if constexpr (WIDE)
                                if (best != INF) As[l] |= (unsigned)first_rp(blp, l, best) << 16;
                        }
                    } else {
                        // the lanes share the scan of l' for the single cell L
                        const Row ql = Q[L];
                        const int mask = mask_of(ql.oh);
                        prm_key best = {PP_INF64, 0, 0};
                        for (int lp = xi - 1 + tl; lp < L; lp += BL) {
                            const Row q = Q[lp];
                            const V last = last_stage(q, ql, mask), g = search ? (V)Gr[lp] : q.g;
                            const V t = g > last ? g : last;
                            prm_key k = {t == INF ? PP_INF64 : (long long)t, lp, 0};
                            if (prm_less(k, best)) best = k;
                        }
                        for (int off = 32; off; off >>= 1) {
                            prm_key ok;
                            ok.v = __shfl_xor(best.v, off);
                            ok.lp = __shfl_xor(best.lp, off);
                            ok.rp = 0;
                            if (prm_less(ok, best)) best = ok;
                        }
                        if constexpr (WIDE) {
                            if (lane == 0) sh.red[wib] = best;
                            __syncthreads();
                            if (tid == 0)
                                for (int w = 1; w < B / 64; ++w)
                                    if (prm_less(sh.red[w], best)) best = sh.red[w];
                        }
                        if (tl == 0) {
                            const bool none = best.v == PP_INF64;
                            Ws[L] = none ? INF : (V)best.v;
                            if constexpr (WIDE) As[L] = none ? 0u : ((unsigned)best.lp | ((unsigned)first_rp(best.lp, L, (V)best.v) << 16));
                            else As[L] = none ? 0u : (unsigned)best.lp;
                        }
                    }
                    sync();  // the g fields (and sh.red) are rewritten by the next state
                }
                sync();  // the records and X are rewritten by the next (r, i)
            }
            __syncthreads();  // the states with more GPUs read these
        }

        // ---- per stage count: the first r with the smallest W (Alg. 3), and its plan
        __threadfence_block();
        __syncthreads();
        for (int xi = 1 + tid; xi <= D; xi += B) {
            V wbest = INF;
            int rbest = 0;
            for (int r = 1; r <= D - xi + 1; ++r) {
                V w = Wt[(size_t)prm_sid(D, xi, r) * L1 + L];
                if (w < wbest) { wbest = w; rbest = r; }
            }
            a.W_out[c * D + xi - 1] = wbest == INF ? PP_INF64 : (long long)wbest;
            int *bo = a.bounds_out + c * tri + xi * (xi - 1) / 2;
            int *ro = a.reps_out + c * tri + xi * (xi - 1) / 2;
            int l = L, n = D, r = rbest;
            for (int s = xi - 1; s >= 0; --s) {
                if (wbest == INF) { bo[s] = 0; ro[s] = 0; continue; }
                bo[s] = l;
                ro[s] = r;
                const size_t at = (size_t)prm_sid(n, s + 1, r) * L1 + l;
                const unsigned arg = At[at];
                const int lp = (int)(arg & 0xffffu);
                if constexpr (WIDE) {
                    n -= r;
                    r = (int)(arg >> 16);
                } else if (s > 0) {
                    // the first r' whose value reaches the cell's (the last stage's term is the same
                    // for all of them)
                    const V v = Wt[at];
                    const int n0 = n - r, nrp = n0 - (s - 1);
                    const double den = r > 1 ? din[n * D1 + r] : 1.0, inv = prm_inv(den), times = 2.0 * (r - 1);
                    const int2 ul = UT[(size_t)(r - 1) * L1 + l], up = UT[(size_t)(r - 1) * L1 + lp];
                    int ral = 0, rap = 0;
                    const int qal = r > 1 ? prm_floor_div(times * PAd[l], den, inv, ral) : 0;
                    const int qap = r > 1 ? prm_floor_div(times * PAd[lp], den, inv, rap) : 0;
                    const V last = ul.x + qal - (up.x + qap) +
                                   (V)((int)M * __popc((unsigned)(up.y & (ul.y - 0x10001)))) + (ral > rap);
                    int rp = 1;
                    for (; rp < nrp; ++rp) {
                        const size_t m = ((size_t)n0 * D1 + rp) * D1 + r;
                        const V x = (int)M * (prm_ceil_div(AF[lp], dfwd[m], prm_inv(dfwd[m])) +
                                              prm_ceil_div(AB[lp], dbwd[m], prm_inv(dbwd[m])));
                        V w = Wt[(size_t)prm_sid(n0, s, rp) * L1 + lp];
                        w = w > x ? w : x;
                        if ((w > last ? w : last) == v) break;
                    }
                    n = n0;
                    r = rp;
                }
                l = lp;
            }
        }
    }
}

__global__ __launch_bounds__(PRM_THREADS) void k_prm(prm_args a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ prm_shared sh;
    if (a.band && a.band[PRM_BAND_PARTS]) return;  // (every candidate has been planned: pp_prm_band.hip)
    const int L = a.L, D = a.D, tid = threadIdx.x, B = blockDim.x;
    const long long M = a.M;
    const int L1 = L + 1, L1p = (L1 + 1) & ~1;
    long long *PF = (long long *)smem, *PB = PF + L1p, *PA = PB + L1p;

    // prefix sums (every workgroup makes its own copy: L is small next to the DP), input checks
    // and the bounds that decide between int32 and int64 values
    if (tid == 0) {
        sh.fault = 0;
        sh.amax_f = sh.amax_b = sh.bmax = 0;
        sh.bmin = ~0ull;
    }
    __syncthreads();
    {
        int fault = 0;
        unsigned long long af = 0, ab = 0, lo = ~0ull, hi = 0;
        for (int l = tid; l < L; l += B) {
            long long x = a.fwd[l], y = a.bwd[l], z = a.alpha[l];
            if (x < 0 || y < 0 || z < 0) fault |= PP_FAULT_NEGATIVE;
            if (l + 1 < L) {
                long long f = a.actf[l], b = a.actb[l];
                if (f < 0 || b < 0) fault |= PP_FAULT_NEGATIVE;
                af = (unsigned long long)f > af ? (unsigned long long)f : af;
                ab = (unsigned long long)b > ab ? (unsigned long long)b : ab;
            }
            if (x >= PP_CAP62 || y >= PP_CAP62 || z >= PP_CAP62) fault |= PP_FAULT_OVERFLOW;
            PF[l + 1] = x; PB[l + 1] = y; PA[l + 1] = z;
        }
        for (int t = tid; t < D * D; t += B)
            if (t / D != t % D) {
                long long b = a.bw[t];
                if (b <= 0) fault |= PP_FAULT_BANDWIDTH;
                lo = (unsigned long long)b < lo ? (unsigned long long)b : lo;
                hi = (unsigned long long)b > hi ? (unsigned long long)b : hi;
            }
        if (fault) atomicOr(&sh.fault, fault);
        atomicMax(&sh.amax_f, af);
        atomicMax(&sh.amax_b, ab);
        atomicMax(&sh.bmax, hi);
        atomicMin(&sh.bmin, lo);
    }
    __syncthreads();
    if (tid == 0 && !sh.fault) {
        long long f = 0, b = 0, al = 0;
        PF[0] = PB[0] = PA[0] = 0;
        for (int l = 1; l <= L; ++l) {
            f += PF[l]; b += PB[l]; al += PA[l];
            // M * (time) and 2 (r-1) * (parameter bytes) must stay far from 2^63
            if (f + b >= PP_CAP62 / (M + 4 * D) || al >= PP_CAP62 / (2 * D)) { sh.fault = PP_FAULT_OVERFLOW; break; }
            PF[l] = f; PB[l] = b; PA[l] = al;
        }
        // int32 values if the largest stage term, the largest channel term and the largest
        // AllReduce remainder all stay below 2^30
        const long long lim = 1ll << 30;
        bool narrow = !sh.fault && M < (1 << 20);
        if (narrow && D > 1) {
            const long long bmin = (long long)sh.bmin;
            narrow = (long long)sh.bmax < lim / D &&
                     cdiv64((long long)sh.amax_f, bmin) + cdiv64((long long)sh.amax_b, bmin) < lim / M &&
                     2 * al / bmin + 1 < lim / 2;
        }
        narrow = narrow && f + b + 2 < lim / (2 * M);
        // (sizes and the multiples of them that are divided must be exact in double arithmetic)
        const unsigned long long exact = 1ull << 53;
        narrow = narrow && D > 1 && sh.amax_f < exact && sh.amax_b < exact && (unsigned long long)al < exact / (2 * D);
        sh.wide = !narrow;
    }
    __syncthreads();
    if (blockIdx.x == 0) {
        if (!sh.fault)
            for (int l = tid; l <= L; l += B) {
                a.pre_out[l] = PF[l];
                a.pre_out[L1 + l] = PB[l];
                a.pre_out[2 * L1 + l] = PA[l];
            }
    }
    if (sh.fault) {
        // nothing can be planned: every (candidate, stage count) is marked as having no plan
        if (tid == 0 && blockIdx.x == 0) pp_raise(a.status, sh.fault);
        for (long long t = (long long)blockIdx.x * B + tid; t < a.N * D; t += (long long)gridDim.x * B)
            a.W_out[t] = PP_INF64;
        return;
    }
    if (sh.wide) prm_run<true>(a, smem, sh);
    else prm_run<false>(a, smem, sh);
}

// Row c = the ordering of lexicographic rank c among all D! (D <= 20).
__global__ __launch_bounds__(256) void k_all_orderings(int D, long long N, int *ord) {
    const long long c = (long long)blockIdx.x * 256 + threadIdx.x;
    if (c >= N) return;
    unsigned long long rem = (unsigned long long)c;
    unsigned used = 0;
    for (int n = 0; n < D; ++n) ord[c * D + n] = pp_unrank_next(D, n, rem, used);
}

// Workspace of pp_plan_replicated.
struct rep_layout {
    size_t slots_at, ord, pre, W, T, bounds, reps, part, total;
    int slots;
};

static rep_layout rep_layout_of(int L, int D, int64_t N) {
    rep_layout w;
    size_t off = 0;
    const size_t tri = (size_t)D * (D + 1) / 2;
    w.slots = (int)(N < 2560 ? N : 2560);  // 10 workgroups of 128 threads per compute unit
    w.slots_at = off; off += pp_align256((size_t)w.slots * prm_slot_bytes(L, D));
    w.ord = off;      off += pp_align256((size_t)N * D * 4);
    w.pre = off;      off += pp_align256((size_t)3 * (L + 1) * 8);
    w.W = off;        off += pp_align256((size_t)N * D * 8);
    w.T = off;        off += pp_align256((size_t)N * D * 8);
    w.bounds = off;   off += pp_align256((size_t)N * tri * 4);
    w.reps = off;     off += pp_align256((size_t)N * tri * 4);
    w.part = off;     off += pp_align256((size_t)PP_PARTS * 16);
    w.total = off;
    return w;
}

static bool rep_sizes_ok(int L, int D, int64_t N, const int32_t *orderings) {
    if (L < 1 || L > PP_MAX_LAYERS || D < 1 || D > 16 || N < 1) return false;
    if (prm_lds_bytes(L, D) > 64 * 1024) return false;
    if (!orderings) {
        int64_t f = 1;
        for (int i = 2; i <= D; ++i) f *= i;  // D <= 16: no overflow
        if (f != N) return false;
    }
    return true;
}

extern "C" size_t pp_workspace_bytes_replicated(int L, int D, int64_t N) {
    if (L < 1 || L > PP_MAX_LAYERS || D < 1 || D > 16 || N < 1) return 0;
    if (prm_lds_bytes(L, D) > 64 * 1024) return 0;
    return rep_layout_of(L, D, N).total;
}

extern "C" int pp_plan_replicated(int L, int D, int64_t N, int M, const int64_t *fwd_us,
                                  const int64_t *bwd_us, const int64_t *act_fwd_bytes,
                                  const int64_t *act_bwd_bytes, const int64_t *alpha_bytes,
                                  const int64_t *bw, const int32_t *orderings, pp_rep_result *out,
                                  int64_t *T_all, int64_t *W_all, int32_t *bounds_all,
                                  int32_t *reps_all, void *workspace, size_t workspace_bytes,
                                  int32_t *status, void *stream) {
    if (!rep_sizes_ok(L, D, N, orderings) || M < 1) return PP_ERR_INVALID_ARG;
    if (!fwd_us || !bwd_us || !act_fwd_bytes || !alpha_bytes || !bw || !out) return PP_ERR_INVALID_ARG;
    const rep_layout lay = rep_layout_of(L, D, N);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < lay.total) return PP_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)workspace;
    const int32_t *ord = orderings;
    if (!ord) {
        int *list = (int *)(base + lay.ord);
        hipLaunchKernelGGL(k_all_orderings, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, D,
                           (long long)N, list);
        if (hipGetLastError() != hipSuccess) return PP_ERR_HIP;
        ord = list;
    }
    const int64_t *actb = act_bwd_bytes ? act_bwd_bytes : act_fwd_bytes;
    int64_t *W = W_all ? W_all : (int64_t *)(base + lay.W);
    int64_t *T = T_all ? T_all : (int64_t *)(base + lay.T);
    int32_t *bounds = bounds_all ? bounds_all : (int32_t *)(base + lay.bounds);
    int32_t *reps = reps_all ? reps_all : (int32_t *)(base + lay.reps);
    int64_t *pre = (int64_t *)(base + lay.pre);

    prm_args a;
    a.L = L; a.D = D; a.M = M; a.N = N;
    a.fwd = (const long long *)fwd_us; a.bwd = (const long long *)bwd_us;
    a.actf = (const long long *)act_fwd_bytes; a.actb = (const long long *)actb;
    a.alpha = (const long long *)alpha_bytes; a.bw = (const long long *)bw;
    a.ord = ord;
    a.scratch = base + lay.slots_at;
    a.slot_bytes = prm_slot_bytes(L, D);
    a.W_out = (long long *)W; a.bounds_out = bounds; a.reps_out = reps;
    a.pre_out = (long long *)pre;
    a.slots = lay.slots;
    a.status = status;
    // the bands' tables lie where the kernels after k_prm write: the partial results, or the times
    const size_t tables = prm_band_bytes(L, D);
    a.band = tables <= lay.total - lay.part ? (int *)(base + lay.part)
             : tables <= lay.bounds - lay.T ? (int *)(base + lay.T) : nullptr;
    if (!prm_band_wanted(a)) a.band = nullptr;
    if (a.band) {
        const int rc = pp_launch_prm_band(a, st);
        if (rc) return rc;
    }
    size_t lds = prm_lds_bytes(L, D);
    a.search = prm_search_lds_bytes(L, D) <= 64 * 1024;
    if (a.search && prm_search_lds_bytes(L, D) > lds) lds = prm_search_lds_bytes(L, D);
    hipLaunchKernelGGL(k_prm, dim3(lay.slots), dim3(PRM_THREADS), lds, st, a);
    if (hipGetLastError() != hipSuccess) return PP_ERR_HIP;
    return pp_launch_rep_makespan(L, D, N, M, pre, pre + (L + 1), pre + 2 * (L + 1), act_fwd_bytes,
                                  actb, bw, ord, bounds, reps, W, T, status, base + lay.part,
                                  out, st);
}
