// Partition DP for 88 < L <= 128: one wavefront per candidate, the rows as in pp_dp_row.h (one lane
// per cell and a search per cell, two chunks of 64 cells side by side).
//
// The rows of the current candidate live in LDS, one private slice per wave, so there are no
// barriers.  The single cell of the last row that is needed is worked out at the end of row S-2,
// from registers.
//
// Row n of a candidate depends only on the first n+1 devices of its ordering.  A wave walks
// a contiguous chunk of candidates and recomputes only the rows from the first position in
// which the ordering differs from the previous candidate's; with all D! orderings in
// lexicographic order most rows are shared.
//
// Reading a plan back is a chain of S-1 dependent lookups, far longer than the arithmetic of
// a candidate that recomputes one or two rows.  So every computed row also leaves its split
// indices (one byte per cell) in an arena in LDS, every finished candidate records which
// arena rows make up its path, and the plans of up to DPR_PENDING finished candidates are read
// back together, one candidate per lane.
//
// What bounds it: instruction issue (107 vector and 85 scalar instructions per row, all told; vector unit
// busy 51 %) and the latency of the searches' LDS reads at three waves per SIMD.  L = 128, S = 8, all 8!
// orderings: 63 us with every (cell, split) pair evaluated from registers, 46 us here; L = 97, S = 11,
// 200 003 sampled orderings, whole call: 1.18 -> 0.93 ms.
#include "pp_common.h"
#include "pp_dp_flat.h"
#include "pp_dp_row.h"
#include "pp_dp_rows.h"

// min over the 64 lanes (uniform result)
__device__ __forceinline__ int wave_min(int v) {
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, true));   // quad_perm:[1,0,3,2]
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, true));   // quad_perm:[2,3,0,1]
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, true));  // row_half_mirror
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, true));  // row_mirror
    return row_imin(row_imin(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                    row_imin(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

__global__ __launch_bounds__(256) void k_dp_rows(dp_rows_args a) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (pp_is_flat(a.g.hdr)) {
        // no channel time depends on the cut position: closed form, here or in the makespan kernel
        if (!dp_flat_deferred(a.g)) dp_flat_body(a.g, smem, a.g.lds_bytes);
        return;
    }
    if (!(pp_vmax(a.g.hdr) < a.g.fit_limit)) {
        dp_generic_body<true>(a.g, smem, *(dp_generic_small *)(smem + dp_generic_rows_bytes(a.g.L)));  // times too large for 32-bit keys
        return;
    }

    constexpr int U = 2, RS = DPR_RS;  // two chunks of 64 cells; row stride: keys in dwords, arena rows in bytes
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int S = a.S, K = a.K, L = a.L, D = a.D;
    const int kmask = (1 << K) - 1;
    // (P[k] << K) - k, k = 0..64 U (P padded with P[L]), shared by the workgroup, with an entry of padding in front
    int *sPk = (int *)smem + 1;
    for (int k = threadIdx.x; k <= 64 * U; k += blockDim.x) sPk[k] = (a.g.p32[k < L ? k : L] << K) - k;
    if (threadIdx.x == 0) sPk[-1] = 0;
    __syncthreads();
    unsigned char *mine = smem + RS * 4 + (size_t)wib * pp_dp_rows_lds_per_wave(S);
    int *rows = (int *)mine;              // [S][RS] keys of the current path's rows
    int *sg = rows + S * RS;              // g and h of the row being computed
    unsigned *sh = (unsigned *)(sg + RS) + 1;
    int *tops = sg + 2 * RS;              // [pending][S] key of cell (n, L)
    unsigned char *arena = (unsigned char *)(tops + DPR_PENDING * S);
    unsigned char *slots = arena + (size_t)dpr_arena_rows(S) * RS;  // [pending][S] arena row of row n
    const int arena_rows = dpr_arena_rows(S);
    const bool stages = a.g.stages != 0;
    const int tri = S * (S + 1) / 2;
    long long *C_out = a.g.C_out;
    int *bounds_out = a.g.bounds_out;
    const int *ord = a.g.ord;

    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + wib;
    const long long c0 = wave * a.chunk;
    const long long c1 = c0 + a.chunk < a.N ? c0 + a.chunk : a.N;
    if (c0 >= c1) return;

    // row 0: one stage holding the first l layers (same for every candidate)
    for (int l = lane; l <= 64 * U; l += 64) rows[l] = sPk[l] + l;
    row_lds_sync();
    const int PLk = sPk[L] + L;
    dp_row r;
    r.g = sg;
    r.h = sh;
    r.PK = sPk;
    r.L = L;
    r.K = K;
    r.kmask = kmask;
    r.strict = row_is_strict(sPk, L, lane);
    r.lane = lane;
    int v_steps = row_first_steps(L, lane);
    const unsigned long long smask = S >= 64 ? ~0ull : ((1ull << S) - 1);
    const int top_lane = (L - 1) & 63;  // the lane of cell L (in the last chunk)

    // finished candidates pend0 .. pend0+pending-1 wait for their plans to be written out;
    // lane q keeps the key of cell (S-1, L) of pending candidate q (-1: its ordering was bad)
    long long pend0 = c0;
    int pending = 0, v_top = 0;
    unsigned long long pairs = 0, nrows = 0;  // work done by this wave
    int arena_used = 0;
    bool fresh = true;  // the arena was emptied: the next candidate must recompute every row
    int v_cur = 0;  // lane n: arena row holding the split indices of row n of the current path
    // lane n: key of cell (n, L) of the current path, i.e. the result for n+1 stages
    int v_tops = PLk;

    // Writes out C and the plans of all pending candidates, one per lane.
    auto flush = [&]() {
        row_lds_sync();
        const bool live = lane < pending;
        const long long cq = pend0 + lane;
        const bool bad = live && v_top < 0;
        if (__ballot(bad) && lane == 0) pp_raise(a.g.status, PP_FAULT_ORDERING);
        // xi = number of stages of the plan read back: S only, or every count 1..S
        for (int xi = stages ? 1 : S; xi <= S; ++xi) {
            int top = v_top;
            if (xi < S && live && !bad) top = tops[lane * S + xi - 1];
            const long long cat = stages ? cq * S + xi - 1 : cq;
            if (live) C_out[cat] = bad ? PP_INF64 : (long long)(top >> K);
            int *bo = bounds_out + (stages ? cq * tri + xi * (xi - 1) / 2 : cq * S);
            int e = L;
            for (int n = xi - 1; n >= 0; --n) {
                if (live) bo[n] = bad ? 0 : e;
                if (n == 0) break;
                // split index stored with cell (n, e): the key itself for the plan's last row
                int nxt = top & kmask;
                if (n < xi - 1 && live && !bad) nxt = arena[(int)slots[lane * S + n] * RS + e] & kmask;
                e = (live && !bad) ? nxt : 0;
            }
        }
        pend0 += pending;
        pending = 0;
        arena_used = 0;
        fresh = true;
    };

    if (S == 1) {
        // a single stage: nothing to compute, C = P[L]
        const int key = rows[L];
        for (long long c = c0; c < c1; ++c) {
            const int d = ord[c];
            const bool bad = a.validate && (d < 0 || d >= D);
            if (lane == pending) v_top = bad ? -1 : key;
            if (++pending == DPR_PENDING) flush();
        }
        if (pending) flush();
        return;
    }

    // Lane n carries device o[n] of the candidate (v_o) and the link index o[n-1]*D + o[n]
    // that row n needs (v_link).
    int v_prev = 0;
    bool have_prev = false;
    int v_o = lane < S ? ord[c0 * S + lane] : 0;

    // Looks at candidate ordering v (previous valid one in v_prev): returns the first row to
    // compute, or -1 if the ordering is not a list of distinct devices below D.
    auto inspect = [&](int v) -> int {
        int p = 0;
        if (have_prev) {
            unsigned long long diff = __ballot(v != v_prev) & smask;
            p = diff ? __builtin_ctzll(diff) : S;
        }
        if (a.validate) {
            bool bad = lane < S && (v < 0 || v >= D);
            for (int q = 0; q + 1 < S; ++q) {
                int oq = __builtin_amdgcn_readlane(v, q);
                bad |= (lane > q && lane < S && oq == v);
            }
            if (__ballot(bad)) return -1;
        }
        // rows below p are reused, so their split indices must still be in the arena
        p = (p > 1 && !fresh) ? p : 1;
        return p < S - 1 ? p : S - 1;  // the last row is always recomputed
    };
    auto links = [&](int v) -> int {
        int up = __shfl_up(v, 1);
        return up * D + v;
    };
    auto fetch_x = [&](int (&x)[U], int link) {
        const int *xp = a.g.x32 + (size_t)link * L;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 64 * u + lane;
            x[u] = xp[k];  // (beyond L: whatever follows the row in the workspace; not used)
        }
    };

    // prio_until[k]: the last candidate with more than prio_left[k] candidates still to do
    // (itself included)
    long long prio_until[3];
    for (int k = 0; k < 3; ++k) prio_until[k] = c1 - 1 - a.prio_left[k];

    // first candidate of the chunk (bad ones are recorded and skipped)
    long long c = c0;
    int first = inspect(v_o);
    while (first < 0) {
        if (lane == pending) v_top = -1;
        if (++pending == DPR_PENDING) flush();
        if (++c >= c1) break;
        v_o = lane < S ? ord[c * S + lane] : 0;
        first = inspect(v_o);
    }
    if (c >= c1) {
        if (pending) flush();
        return;
    }
    int v_link = links(v_o);
    int xk[U];
    fetch_x(xk, __builtin_amdgcn_readlane(v_link, first));

    for (;;) {
        // c is a valid candidate whose rows first..S-1 are to be computed; xk holds (or is
        // about to receive) the channel keys of row `first`
        fresh = false;
        // Of the waves that share a SIMD the one with more of its chunk still to do issues
        // first, so that they finish together and none runs alone at the end (levels from
        // thresholds worked out once: a division here costs as much as a tenth of a row).
        if (c <= prio_until[2]) __builtin_amdgcn_s_setprio(3);
        else if (c <= prio_until[1]) __builtin_amdgcn_s_setprio(2);
        else if (c <= prio_until[0]) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
        const bool more = c + 1 < c1;
        int v_on = (more && lane < S) ? ord[(c + 1) * S + lane] : 0;
        int first_n = -2, v_link_n = 0;  // next candidate: -2 none, -1 bad ordering
        bool flush_after = false;

        // candidate finished with key `top` in cell (S-1, L): remember it and the arena rows of
        // its path
        auto finish_candidate = [&](int top) __attribute__((always_inline)) {
            if (lane == pending) v_top = top;
            if (lane < S) slots[pending * S + lane] = (unsigned char)v_cur;
            if (stages && lane < S) tops[pending * S + lane] = v_tops;
            ++pending;
        };

        // One DP row.  xc holds this row's channel keys; the keys of the row computed next are
        // fetched into xf while this one is computed.  After the candidate's last row that is
        // the first row of the next candidate (looked at here), or, if there is none, this
        // row's keys once more.
        auto row = [&](int n, int (&xc)[U], int (&xf)[U]) __attribute__((always_inline)) {
            int next_link = __builtin_amdgcn_readlane(v_link, n + 1 < S ? n + 1 : n);
            // the candidate ends with this row: the last row itself, or row S-2 with cell
            // (S-1, L) worked out at its end
            const bool fused = n == S - 2;
            int xl[U];
            if (fused) {
                const int *xp = a.g.x32 + (size_t)next_link * L;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int l = 64 * u + lane + 1;
                    xl[u] = xp[l];
                }
            }
            if ((n == S - 1 || fused) && more) {
                v_prev = v_o;
                have_prev = true;
                first_n = inspect(v_on);
                if (first_n >= 0) {
                    // rows first_n..S-2 need arena rows (and so does this row, if it is row
                    // S-2); one more pending candidate needs a lane
                    if (arena_used + (fused ? 1 : 0) + (S - 1 - first_n) > arena_rows ||
                        pending + 2 > DPR_PENDING) {
                        flush_after = true;
                        first_n = 1;
                    }
                    v_link_n = links(v_on);
                    next_link = __builtin_amdgcn_readlane(v_link_n, first_n);
                }
            }
            fetch_x(xf, next_link);

            r.W = rows + (n - 1) * RS;
            if (n < S - 1) {
                r.out = rows + n * RS;
                r.n = n;
                r.steps = __builtin_amdgcn_readlane(v_steps, n);
                r.carry = PP_INF32;
                r.again = false;
                int w[U];
                row_build<U>(r, 0, xc, w);
                row_lds_sync();
                row_search<U>(r, 0, w);
                pairs += (unsigned long long)((L - n) * (r.steps + 1));
                ++nrows;
                if (r.again && lane == n && v_steps < K) ++v_steps;
                const int slot = arena_used++;
                const int top_n = __builtin_amdgcn_readlane(w[U - 1], top_lane);
                if (lane == n) { v_cur = slot; v_tops = top_n; }
                // low byte of the key: the split index in its low K <= 7 bits
                unsigned char *arow = arena + slot * RS + lane + 1;
#pragma unroll
                for (int u = 0; u < U; ++u) arow[64 * u] = (unsigned char)w[u];
                if (fused) {
                    // cell (S-1, L), the only cell of the last row that is needed, from row S-2's
                    // cells while they are in registers
                    int m = PP_INF32;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int l = 64 * u + lane + 1;
                        const int xk2 = (int)((unsigned)xl[u] << K) | l, wk = (w[u] & ~kmask) | l;
                        const int t = row_imax(row_imax(wk, xk2), PLk - sPk[l]);
                        m = l < L ? row_imin(m, t) : m;
                    }
                    const int top = wave_min(m);
                    pairs += (unsigned long long)(L - (S - 1));
                    ++nrows;
                    finish_candidate(top);
                }
                row_lds_sync();
            } else {
                // only W[S-1][L] is needed of the last row
                int m = PP_INF32;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int k = 64 * u + lane;
                    const int xk2 = (int)((unsigned)xc[u] << K) | k, wk = (r.W[k] & ~kmask) | k;
                    const int t = row_imax(row_imax(wk, xk2), PLk - sPk[k]);
                    m = (k >= n && k < L) ? row_imin(m, t) : m;
                }
                pairs += (unsigned long long)(L - n);
                ++nrows;
                finish_candidate(wave_min(m));
            }
        };
        // rows alternate between the two key buffers, so that no row has to copy them; only a
        // candidate with an odd number of rows moves the last fetch into xk once
        int xn[U];
        // (the last row is a row of its own only when no other row is computed)
        const int end = first <= S - 2 ? S - 1 : S;
        for (int n = first;;) {
            row(n, xk, xn);
            if (++n >= end) {
#pragma unroll
                for (int u = 0; u < U; ++u) xk[u] = xn[u];
                break;
            }
            row(n, xn, xk);
            if (++n >= end) break;
        }

        if (flush_after) flush();
        // bad orderings after this candidate are recorded and skipped
        while (first_n == -1) {
            if (lane == pending) v_top = -1;
            if (++pending == DPR_PENDING) flush();
            ++c;
            first_n = -2;
            if (c + 1 < c1) {
                v_on = lane < S ? ord[(c + 1) * S + lane] : 0;
                first_n = inspect(v_on);  // compared with the last valid candidate
                if (first_n >= 0) {
                    if (arena_used + (S - 1 - first_n) > arena_rows || pending + 2 > DPR_PENDING) {
                        flush();
                        first_n = 1;
                    }
                    v_link_n = links(v_on);
                    fetch_x(xk, __builtin_amdgcn_readlane(v_link_n, first_n));
                }
            }
        }
        if (first_n < 0) break;  // no candidate left
        ++c;
        v_o = v_on;
        v_link = v_link_n;
        first = first_n;
    }
    if (pending) flush();
    if (lane == 0) pp_count_work(a.g.hdr, pairs, nrows, (unsigned)wave);
}

int pp_launch_dp_rows(const dp_rows_args &a, int grid, int wpb, hipStream_t st) {
    size_t lds = (size_t)DPR_RS * 4 + (size_t)wpb * pp_dp_rows_lds_per_wave(a.S);
    const size_t generic = dp_generic_lds_bytes(a.L);  // the int64 fallback's rows
    if (lds < generic) lds = generic;
    const size_t flat = pp_flat_lds_wanted(a.L, a.D, a.S, wpb);  // the closed-form body's tables
    if (lds < flat) lds = flat;
    dp_rows_args b = a;
    b.g.lds_bytes = lds;
    hipLaunchKernelGGL(k_dp_rows, dim3(grid), dim3(64 * wpb), lds, st, b);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
