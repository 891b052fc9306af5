// Partition DP for 128 < L <= 2048 with 32-bit keys: one wavefront per candidate, the rows as in
// pp_dp_row.h, up to four chunks of 64 cells side by side.
//
// What bounds it: the latency of the searches' LDS reads, then instruction issue (vector unit busy
// 63 % at L = 1024, where the LDS holds three waves per SIMD; four chunks side by side give each
// wave four reads in flight).  About 37 K vector instructions per candidate at L = 1024, S = 32,
// against 125 K when every (cell, split) pair up to an exact early exit was evaluated: 2^20
// candidates 275 -> 98 ms; L = 300, S = 16, 15 751 representatives 297 -> 203 us.  Where links bind at
// every cut (1.25 GB/s, activations that shrink; DP alone): L = 1024, S = 16 522 -> 280 us for 500
// candidates, L = 300, S = 16 176 -> 143 us for 2 777.  (One lane per row
// and one step per cell with a monotone queue was measured too: 345 ms at L = 1024, a serial chain of
// LDS trips per cell.)
//
// Only candidates that the bands (pp_dp_band.h) have left come here where those are tried.
//
// Per wave in LDS: two rows of keys (the row being read, rewritten in place as g, and the row
// being produced) and h.  Split indices go to a per-wave table in global memory while the next
// row's g is built (coalesced), and the plan is read back from there with cache-bypassing
// loads.  Waves are persistent and walk candidates wave, wave + nwaves, ...; where groups of
// candidates are the same problem (pp_share.hip) a wave instead takes a run of consecutive
// entries of the sorted list of representatives, keeps every row it computes in the workspace
// and starts each representative at the first row its predecessor does not share.
#include "pp_common.h"
#include "pp_dp_flat.h"
#include "pp_dp_generic.h"
#include "pp_dp_row.h"

// Rows in which more than one split in ROW_FALLS is undercut by a later one are searched with minima that end
// at the cell (row_jump).  DP alone against a kernel that evaluates all (cell, split) pairs up to an early
// exit, thresholds of no row / L/4 / L/16 / L/64 / every row with one: links that bind everywhere (1.25 GB/s,
// activations that shrink) L = 300, S = 16 0.54x / 0.53x / 1.23x / 1.22x / 1.23x; channel times of about a
// stage's, in no order, L = 192, S = 64 0.81x / 0.98x / 1.13x / 1.23x / 1.23x, L = 1024, S = 16 1.88x / 1.88x /
// 2.02x / 1.88x / 1.75x; times that seldom bind, L = 1024, S = 32 2.18x / 2.17x / 2.17x / 2.16x / 1.83x.
#define ROW_FALLS 16
struct dp_big_args {
    int NC;      // chunks of 64 cells: ceil(L / 64)
    int waves;   // working waves (each owns one backtrack table)
    size_t arg_stride;  // entries of one wave's backtrack table: S * Lp
    // non-NULL: if the workspace header says so, walk this list of representatives (one per
    // group of candidates with the same DP, see pp_share.hip) instead of all candidates: every
    // wave a run of neighbours, which share their first links and so their first rows (keys:
    // the key of every candidate; rows: room for row_slots saved rows of Lp + 4 keys)
    // pend: the representatives the bands have left, the list that is really walked
    const int *reps, *pend, *keys, *start;
    int *rows;
    long long row_slots;  // rows of Lp + 4 keys the area `rows` holds
    dp_args g;
};

// Where the split of cell k of a row stands in its row of the backtrack table: the four chunks of a
// whole group of 256 cells lane by lane (one store of 8 bytes per lane), the rest cell by cell.
__device__ __forceinline__ int big_arg_at(int k, int Lp) {
    return k < (Lp & ~255) ? (k & ~255) | (k & 63) << 2 | (k >> 6 & 3) : k;
}

// The chunks c0 .. c0 + 64 U - 1 of a row being built (c0 a multiple of 256).  xv: the link's times;
// arow: where the previous row's split indices go (NULL: nowhere).
template <int U>
__device__ __forceinline__ void big_build(dp_row &r, int c0, const int (&xv)[4], unsigned short *arow) {
    int w[U];
    row_build<U>(r, c0, xv, w);
    if (!arow) return;
    if (U == 4) {
        const unsigned lo = (unsigned)(w[0] & r.kmask) | (unsigned)(w[U > 1 ? 1 : 0] & r.kmask) << 16;
        const unsigned hi = (unsigned)(w[U > 2 ? 2 : 0] & r.kmask) | (unsigned)(w[U > 3 ? 3 : 0] & r.kmask) << 16;
        *(uint2 *)(arow + c0 + 4 * r.lane) = make_uint2(lo, hi);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) arow[c0 + 64 * u + r.lane] = (unsigned short)(w[u] & r.kmask);
    }
}

__global__ __launch_bounds__(256, 4) void k_dp_big(dp_big_args b) {
    extern __shared__ __align__(16) unsigned char smem[];
    const dp_args &a = b.g;
    if (pp_is_flat(a.hdr)) {
        // no channel time depends on the cut position: closed form, here or in the makespan kernel
        if (!dp_flat_deferred(a)) dp_flat_body(a, smem, a.lds_bytes);
        return;
    }
    if (!(pp_vmax(a.hdr) < a.fit_limit)) {
        dp_generic_body<true>(a, smem, *(dp_generic_small *)(smem + dp_generic_rows_bytes(a.L)));  // times too large for 32-bit keys
        return;
    }
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wpb = blockDim.x >> 6;
    const int S = a.S, K = a.K, L = a.L, D = a.D;
    const int Lp = 64 * b.NC, RS = Lp + 4;
    const int kmask = (1 << K) - 1;
    // (P[k] << K) - k, k = 0..Lp (P padded with P[L]); this wave's two rows and h.  Every array has
    // an entry of padding in front (index -1).
    int *sPk = (int *)smem + 1;
    int *bufA = sPk + RS + (size_t)wib * 3 * RS;
    int *bufB = bufA + RS;
    const long long wave = (long long)blockIdx.x * wpb + wib;

    unsigned short *arg = a.arg + (size_t)wave * b.arg_stride;
    unsigned long long pairs = 0, nrows = 0;
    const int tri = S * (S + 1) / 2;

    // Which candidates this wave takes: every waves-th one, or a run of consecutive entries of a
    // list the preparation left (pp_share.hip): the sorted representatives where candidates
    // share their DP, or candidates sorted by their first devices (less those whose plans are
    // there already).  Neighbours in a list
    // share their first rows; the wave keeps the rows that can be shared (all of them, or the
    // first kdev - 1) in its slice of the workspace.
    const bool listed = b.reps != NULL && a.hdr->share_active != 0;
    const bool sorted = b.reps != NULL && !listed && a.hdr->share_sorted != 0;
    // main part: entries r_begin, r_begin + r_step, ... (n_main of them); then, where candidates
    // share their DP, this wave's share of the candidates with a bad ordering that follow the
    // sorted representatives in the list (n_tail entries t_begin, t_begin + waves, ...)
    long long r_begin = wave, r_step = b.waves, nsorted = 0, t_begin = 0, n_tail = 0;
    const bool working = wave < b.waves;
    long long n_main = working && wave < a.N ? (a.N - wave + b.waves - 1) / b.waves : 0;
    unsigned pw = 1;  // lane n = 1..S-1: (classes)^(S-1-n), the weight of the key's digit n
    int keep_rows = 0;  // rows 1..keep_rows are saved
    if (listed) {
        // runs of about equal work, cut by the preparation
        const long long total = a.hdr->share_nreps, nch = a.hdr->share_nchunks;
        nsorted = a.hdr->share_nsorted;
        keep_rows = S - 2 > 0 ? S - 2 : 0;
        r_begin = wave < nch ? b.start[wave] : 0;
        n_main = wave < nch ? b.start[wave + 1] - r_begin : 0;
        r_step = 1;
        t_begin = nsorted + wave;
        n_tail = working && t_begin < total ? (total - t_begin + b.waves - 1) / b.waves : 0;
        const unsigned nc = a.hdr->share_nc;
        for (int n = lane + 1; n < S; ++n) pw *= nc;
    } else if (sorted) {
        const long long todo = a.hdr->share_nsorted;  // (what the bands have left)
        keep_rows = (int)a.hdr->share_kdev - 1;
        keep_rows = keep_rows < S - 2 ? keep_rows : S - 2;
        keep_rows = keep_rows > 0 ? keep_rows : 0;
        long long nw = b.row_slots / (keep_rows > 0 ? keep_rows : 1);  // waves whose rows fit the area
        nw = nw < b.waves ? nw : b.waves;
        nw = nw > 1 ? nw : 1;
        const long long chunk = (todo + nw - 1) / nw;
        r_begin = wave * chunk;
        n_main = r_begin < todo ? (r_begin + chunk < todo ? chunk : todo - r_begin) : 0;
        r_step = 1;
    }
    const long long n_items = n_main + n_tail;
    if (__syncthreads_and(n_items == 0)) return;
    for (int k = threadIdx.x; k <= Lp; k += blockDim.x) sPk[k] = (a.p32[k < L ? k : L] << K) - k;
    if (threadIdx.x == 0) sPk[-1] = 0;
    __syncthreads();
    if (!n_items) return;
    dp_row row;
    row.h = (unsigned *)(bufB + RS);
    row.PK = sPk;
    row.L = L;
    row.K = K;
    row.kmask = kmask;
    row.lane = lane;
    row_begin(row);
    int v_steps = row_first_steps(L, lane);  // lane n: steps of a search in row n
    auto entry = [&](long long i) { return i < n_main ? r_begin + i * r_step : t_begin + (i - n_main) * b.waves; };
    // (row n >= 1 of this wave's slice at save + (n - 1) RS)
    int *save = b.rows + (size_t)((listed || sorted) && n_main ? wave : 0) * keep_rows * RS;
    int prev_key = -1, prev_o = -1;
    int v_tops = 0;  // lane n keeps W[n][L] (with its split index) for the stage-count search
    int *cur = bufA, *nxt = bufB;
    // A candidate's index, key and devices come from memory through a chain of loads (list
    // entry, then key and ordering): they are fetched one candidate ahead.
    auto fetch = [&](long long i, long long &c, int &key, int &v_o) {
        c = 0; key = -1; v_o = 0;
        if (i >= n_items) return;
        const long long r = entry(i);
        c = listed ? (i < n_main ? b.pend[r] : pp_share_at(a.hdr, b.reps, a.N, r)) : sorted ? b.reps[r] : r;
        if (listed && i < n_main) key = b.keys[c];
        v_o = lane < S ? a.ord[c * S + lane] : 0;
    };
    long long c_next;
    int key_next, v_o_next;
    fetch(0, c_next, key_next, v_o_next);
    for (long long i = 0; i < n_items; ++i) {
        const long long c = c_next;
        const int v_o = v_o_next;
        // rows 1..p of the previous candidate are this one's too: its key has the same first p
        // digits (equal links give equal rows), or its first p + 1 devices are the same
        int p = 0;
        const int key = key_next;
        fetch(i + 1, c_next, key_next, v_o_next);
        if (listed && i < n_main) {
            if (prev_key >= 0) {
                const bool differ = lane >= 1 && lane < S && (unsigned)key / pw != (unsigned)prev_key / pw;
                const unsigned long long m = __ballot(differ);
                p = m ? __builtin_ctzll(m) - 1 : S - 2;
                p = p < S - 2 ? p : S - 2;
                p = p > 0 ? p : 0;
            }
        }
        prev_key = key;
        // ordering: lane n holds device o[n]
        bool bad = false;
        if (a.validate) {
            bad = lane < S && (v_o < 0 || v_o >= D);
            for (int q = 0; q + 1 < S; ++q) {
                int oq = __builtin_amdgcn_readlane(v_o, q);
                bad |= (lane > q && lane < S && oq == v_o);
            }
        }
        if (__ballot(bad)) {
            if (lane == 0) pp_raise(a.status, PP_FAULT_ORDERING);
            if (a.stages) {
                if (lane < S) a.C_out[c * S + lane] = PP_INF64;
                for (int n = lane; n < tri; n += 64) a.bounds_out[c * tri + n] = 0;
            } else {
                if (lane == 0) a.C_out[c] = PP_INF64;
                if (lane < S) a.bounds_out[c * S + lane] = 0;
            }
            prev_key = -1;  // (the next candidate starts from row 0)
            prev_o = -1;
            continue;
        }
        if (sorted) {
            // (prev_o: the previous candidate's device in this lane, -1 if there is none)
            const unsigned long long m = __ballot(lane < S && v_o != prev_o);
            p = m ? __builtin_ctzll(m) - 1 : S - 2;
            p = p < keep_rows ? p : keep_rows;
            p = p > 0 ? p : 0;
            prev_o = v_o;
        }
        const int v_link = __shfl_up(v_o, 1) * D + v_o;

        int top = 0;
        if (p == 0) {
            // row 0: one stage holding the first l layers
            for (int l = lane; l <= Lp; l += 64) cur[l] = l ? sPk[l] + l : PP_INF32;
            row_lds_sync();
            top = cur[L];  // S == 1: C = P[L]
            v_tops = top;
        } else {
            // row p as this wave left it (stored by other lanes of the wave: wait for the
            // stores, then read past the L1 cache)
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            const int *from = save + (size_t)(p - 1) * RS;
            for (int l = lane; l <= Lp; l += 64)
                cur[l] = __hip_atomic_load(from + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            row_lds_sync();
        }

        // the links' times are requested 256 splits ahead (from row to row as well)
        const int c_last = (Lp - 1) & ~255;  // first split of the last group of four chunks
        int xv[4], xn[4];
        auto fetch_x = [&](int (&x)[4], const int *xrow, int c0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = c0 + 64 * u + lane;
                x[u] = k < L ? xrow[k] : 0;
            }
        };
        fetch_x(xv, a.x32 + (size_t)__builtin_amdgcn_readlane(v_link, p + 1 < S ? p + 1 : p) * L, c_last);
        for (int n = p + 1; n < S; ++n) {
            // The previous row's split indices (the low key bits) go to the backtrack table.
            unsigned short *arow = n >= 2 ? arg + (size_t)(n - 1) * Lp : NULL;
            const int *xrow = a.x32 + (size_t)__builtin_amdgcn_readlane(v_link, n) * L;
            const int *xnext = a.x32 + (size_t)__builtin_amdgcn_readlane(v_link, n + 1 < S ? n + 1 : n) * L;
            // (the times of the splits c0 .. c0 + 255 of this row, or the last ones of the next row)
            auto fetch_from = [&](int c0) {
                const bool here = c0 >= 0;
                fetch_x(xn, here ? xrow : xnext, here ? c0 : c_last);
            };
            if (n < S - 1) {
                row.W = row.g = cur;
                row.out = nxt;
                row.n = n;
                row.steps = __builtin_amdgcn_readlane(v_steps, n);
                row.carry = PP_INF32;
                row.again = 0;
                row.falls = 0;
                for (int c0 = c_last; c0 >= 0; c0 -= 256) {
                    const int left = (Lp - c0) >> 6;
                    if (left >= 4) big_build<4>(row, c0, xv, arow);
                    else if (left == 3) big_build<3>(row, c0, xv, arow);
                    else if (left == 2) big_build<2>(row, c0, xv, arow);
                    else big_build<1>(row, c0, xv, arow);
                    // (after the stores, so that the wait for the times does not have to be one for
                    // younger stores)
                    fetch_from(c0 - 256);
#pragma unroll
                    for (int u = 0; u < 4; ++u) xv[u] = xn[u];
                }
                row_lds_sync();
                if (row.falls * ROW_FALLS > L) {
                    row_tables(row);
                    int trips = 0;  // of 64 cells
                    for (int c0 = c_last; c0 >= 0; c0 -= 256) {
                        const int left = (Lp - c0) >> 6;
                        if (left >= 4) trips += 4 * row_jump<4>(row, c0);
                        else if (left == 3) trips += 3 * row_jump<3>(row, c0);
                        else if (left == 2) trips += 2 * row_jump<2>(row, c0);
                        else trips += row_jump<1>(row, c0);
                    }
                    pairs += (unsigned long long)(64 * trips);
                } else {
                    for (int c0 = 0; c0 < Lp; c0 += 256) {
                        const int left = (Lp - c0) >> 6;
                        if (left >= 4) { int w[4]; row_search<4>(row, c0, w); }
                        else if (left == 3) { int w[3]; row_search<3>(row, c0, w); }
                        else if (left == 2) { int w[2]; row_search<2>(row, c0, w); }
                        else { int w[1]; row_search<1>(row, c0, w); }
                    }
                    pairs += (unsigned long long)(L - n) * (unsigned)(row.steps + 1) + (unsigned)(64 * row.again * row.steps);
                }
                if (row.again && lane == n && v_steps < K) ++v_steps;
                row_lds_sync();
                int *t = cur; cur = nxt; nxt = t;
                const int top_n = cur[L];
                if (lane == n) v_tops = top_n;
                if (n <= keep_rows) {
                    // kept for the next candidate of the run
                    int *to = save + (size_t)(n - 1) * RS;
                    for (int l = lane; l <= Lp; l += 64) to[l] = cur[l];
                }
            } else {
                // only W[S-1][L] is needed of the last row
                const int PL = sPk[L] + L;
                int v = PP_INF32;
                for (int c0 = c_last; c0 >= 0; c0 -= 256) {
                    fetch_from(c0 - 256);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int k = c0 + 64 * u + lane;
                        if (k >= L) continue;
                        const int w = cur[k];
                        if (arow) arow[big_arg_at(k, Lp)] = (unsigned short)(w & kmask);
                        const int xk = (int)((unsigned)xv[u] << K) | k, wk = (w & ~kmask) | k;
                        const int t = row_imax(row_imax(wk, xk), PL - sPk[k]);
                        v = k >= n ? row_imin(v, t) : v;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) xv[u] = xn[u];
                }
                for (int off = 32; off; off >>= 1) v = row_imin(v, __shfl_xor(v, off));
                top = v;
                if (lane == n) v_tops = v;
                pairs += (unsigned long long)(L - n);
            }
            ++nrows;
        }

        // plan: every lane follows the same chain through the backtrack table, lane n keeps
        // bound n.  The table was written by other lanes of this wave: wait for the stores,
        // then read past the L1 cache (which may hold lines of an earlier candidate).
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        if (a.stages) {
            // lane xi-1 follows its own chain from (xi-1, L): the plan with xi stages
            if (lane < S) {
                a.C_out[c * S + lane] = (long long)(v_tops >> K);
                int *bo = a.bounds_out + c * tri + lane * (lane + 1) / 2;
                int e = L;
                for (int m = lane; m >= 1; --m) {
                    bo[m] = e;
                    if (m == lane) {
                        e = v_tops & kmask;
                        e = e < Lp ? e : Lp - 1;  // stays inside the table whatever the data
                    } else {
                        const size_t at = (size_t)m * Lp + big_arg_at(e, Lp);
                        const unsigned *word = (const unsigned *)(arg + (at & ~(size_t)1));
                        unsigned w2 = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        e = (int)((at & 1) ? (w2 >> 16) : (w2 & 0xffffu));
                    }
                }
                bo[0] = e;
            }
            continue;
        }
        int e = L, mine = 0;
        for (int m = S - 1; m >= 1; --m) {
            if (lane == m) mine = e;
            if (m == S - 1) {
                e = top & kmask;
            } else {
                const size_t at = (size_t)m * Lp + big_arg_at(e, Lp);
                const unsigned *word = (const unsigned *)(arg + (at & ~(size_t)1));
                unsigned w2 = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                e = (int)((at & 1) ? (w2 >> 16) : (w2 & 0xffffu));
            }
        }
        if (lane == 0) { mine = e; a.C_out[c] = (long long)(top >> K); }
        if (lane < S) a.bounds_out[c * S + lane] = mine;
    }
    if (lane == 0) pp_count_work(a.hdr, pairs, nrows, (unsigned)wave);
}

// LDS of a workgroup and waves per workgroup for this shape (0 if it does not fit).
static size_t big_lds(int L, int D, int S, int &wpb) {
    const int Lp = 64 * ((L + 63) / 64), RS = Lp + 4;
    wpb = 4;  // waves per workgroup: table + two rows and h per wave within 64 KiB of LDS
    while (wpb > 1 && (size_t)(1 + 3 * wpb) * RS * 4 > 64 * 1024) wpb >>= 1;
    size_t lds = (size_t)(1 + 3 * wpb) * RS * 4;
    const size_t generic = dp_generic_lds_bytes(L);  // the int64 fallback's rows
    if (lds < generic) lds = generic;
    const size_t flat = pp_flat_lds_wanted(L, D, S, wpb);  // the closed-form body's tables
    if (lds < flat) lds = flat;
    return lds > 64 * 1024 ? 0 : lds;
}

int pp_dp_big_waves(int L, int D, int S, int max_waves, int cus) {
    int wpb;
    const size_t lds = big_lds(L, D, S, wpb);
    if (!lds) return 1;
    // resident waves: 4 per SIMD by registers, and what 160 KiB of LDS per CU allow
    // (given out in pieces of 1280 bytes)
    long long per_cu = (long long)(160 * 1024 / ((lds + 1279) / 1280 * 1280)) * wpb;
    if (per_cu > 16) per_cu = 16;
    if (per_cu < 1) per_cu = 1;
    long long waves = per_cu * cus;
    if (waves > max_waves) waves = max_waves;
    return (int)(waves < 1 ? 1 : waves);
}

int pp_launch_dp_big(const dp_args &g, int max_waves, int cus, const pp_share_list *list,
                     hipStream_t st) {
    dp_big_args b;
    b.g = g;
    b.reps = list ? list->reps : NULL;
    b.pend = list ? list->pend : NULL;
    b.keys = list ? list->keys : NULL;
    b.start = list ? list->start : NULL;
    b.rows = list ? list->rows : NULL;
    b.row_slots = list ? list->row_slots : 0;
    b.NC = (g.L + 63) / 64;
    b.arg_stride = (size_t)g.S * 64 * b.NC;
    int wpb;
    const size_t lds = big_lds(g.L, g.D, g.S, wpb);
    if (!lds) return PP_ERR_INVALID_ARG;
    b.g.lds_bytes = lds;
    const long long waves = pp_dp_big_waves(g.L, g.D, g.S, max_waves, cus);
    b.waves = (int)waves;
    const int grid = (int)((waves + wpb - 1) / wpb);
    b.g.nblocks = g.nblocks < grid ? g.nblocks : grid;
    hipLaunchKernelGGL(k_dp_big, dim3(grid), dim3(64 * wpb), lds, st, b);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
