// Partition DP for 88 < L <= 128 and lists long enough to fill the chip: one wavefront per candidate, one
// lane per cell (two chunks of 64 side by side) and a binary search per cell.
//
// Recursion for W(l, xi, r, i) of Sec. IV-B / the PRM listing with one replica per stage:
//   W[n][l] = min_{n<=k<l} max(g[k], P[l] - P[k]),   g[k] = max(W[n-1][k], X_n[k]),
// lowest minimising k kept; cells and splits are 32-bit keys (time << K) | k.
//
// With G(j) = min_{j<k<l} g[k] (infinite for j = l - 1) a split j is alive iff P[l] - P[j] <= G(j).  G rises
// with j and P[l] - P[j] falls, so the alive splits are those from some j* on.  A split left of j* costs more
// than the one whose g its difference exceeds; among the alive ones no difference exceeds a later g, so
//   W[n][l] = min(G(j*), max(g[j*], P[l] - P[j*])),
// and with keys for times this is the lowest split too (P strictly rising; where layers of length zero make
// lower splits with j*'s P tie, the lowest of their run is looked up).  j* is found from l - 1 downwards by
// powers of two, G growing along: T[s][k] = min g[k+1 .. k+2^s] gives the minimum over a jump.  The tables
// for s = 0 .. steps - 1 take a pass each over the row (two passes per trip to LDS) and lie in the rows that
// are computed after this one.
//
// The minima end at the cell itself, so the work does not depend on where the links bind.  (Minima over the
// whole row, one table, and a walk over the splits wherever a later g undercuts the cell's, as pp_dp_row.h
// has it, took 46 us where this takes 47 - L = 128, S = 8, all 8! orderings, channel times that seldom bind;
// 63 us with all pairs from registers - but with activations that shrink from layer to layer and 1.25 GB/s
// links 341 us for the whole search, against 90 us with all pairs and 78 us here; L = 89, S = 16, 24 000
// orderings 2.4 ms, 0.30 ms, and the tiled kernel's 0.30 ms by pp_dp_tiles.)
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
// What bounds it: instruction issue (187 vector and 154 scalar instructions per row, all told; vector unit
// busy 67 %) and the latency of a row's two chains through LDS, the tables' and the search's: a row takes
// 5 200 clocks with four waves per SIMD.  L = 97, S = 11, 200 003 sampled orderings, whole
// call: 1.18 ms with all pairs, 0.96 ms here.
#include "pp_common.h"
#include "pp_dp_band.h"
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

// One row n (xv: the link's times at the splits 64 u + lane + 1): W[n] to row n of the wave's rows, and to w.
// Returns the number of rounds the searches took.
struct rows_row {
    int *rows;      // the wave's rows, RS entries each
    const int *PK;  // (P[k] << K) - k, k = 0 .. 128
    int RS, L, K, kmask, lane;
    bool strict;    // no layer has length zero
    const unsigned char *run;  // the first split of every split's run of equal P, k = 0 .. 127
    // of the cells 64 u + lane + 1: P, and the entry of PK of their last split (the cells beyond L repeat L)
    unsigned Pl[2];
    int last[2];
};
__device__ __forceinline__ int rows_compute(const rows_row &r, int n, int steps, const int (&xv)[2], int (&w)[2]) {
    const int lane = r.lane, RS = r.RS;
    int *T = r.rows + n * RS;
    // T[s RS + k] = min g[k + 1 .. k + 2^s] (what a search in front of split k + 2^s asks for), 0 for k < n.
    // (Only entries whose whole range lies below L are read back, whatever the others hold.)
    int m[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int k = 64 * u + lane + 1;
        m[u] = row_imax((T[k - RS] & ~r.kmask) | k, (int)((unsigned)xv[u] << r.K) | k);
    }
    const int g_n = __builtin_amdgcn_readlane(m[0], n - 1);
    m[0] = lane >= n ? m[0] : 0;
    T += lane;
#pragma unroll
    for (int u = 0; u < 2; ++u) T[64 * u] = m[u];
    row_lds_sync();
    int *t = T;
    for (int s = 0, by = 1; s + 1 < steps; s += 2, by *= 4) {
        int x[2], y[2], z[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) { x[u] = t[by + 64 * u]; y[u] = t[2 * by + 64 * u]; z[u] = t[3 * by + 64 * u]; }
        t += RS;
#pragma unroll
        for (int u = 0; u < 2; ++u) { x[u] = row_imin(m[u], x[u]); m[u] = row_imin(row_imin(x[u], y[u]), z[u]); }
#pragma unroll
        for (int u = 0; u < 2; ++u) t[64 * u] = x[u];
        t += RS;
        row_lds_sync();  // (other lanes' spills before this table's entries)
        if (s + 2 < steps) {
#pragma unroll
            for (int u = 0; u < 2; ++u) t[64 * u] = m[u];
        }
        row_lds_sync();
    }
    // at[u]: (address of) the entry of P of the split each cell has got back to, low[u]: min g over the
    // splits right of it
    const int pk0 = row_addr(r.PK), to_t = row_addr(T - lane) - pk0, reach = (4 << steps) - 4;
    int at[2];
    unsigned low[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) { at[u] = r.last[u]; low[u] = PP_INF32; }
    int rounds = 0;
    for (bool more = true; more; ++rounds) {
        int from[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) from[u] = at[u];
        for (int by = 2 << steps, to = to_t + 4 * (steps - 1) * RS; by >= 4; by >>= 1, to -= 4 * RS) {
            int j[2];
            unsigned p[2], q[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) { j[u] = at[u] - by; p[u] = row_at(j[u]); q[u] = row_at(j[u] + to); }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const unsigned h = q[u] < low[u] ? q[u] : low[u];
                const bool back = r.Pl[u] - p[u] < h;  // (equal keys cannot be: the split's index is in them)
                at[u] = back ? j[u] : at[u];
                low[u] = back ? h : low[u];
            }
        }
        bool whole = false;
#pragma unroll
        for (int u = 0; u < 2; ++u) whole |= at[u] == from[u] - reach;
        more = __ballot(whole) != 0;
    }
    unsigned g[2], p[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) { g[u] = row_at(at[u] + to_t - 4); p[u] = row_at(at[u]); }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int d = (int)(r.Pl[u] - p[u]), gk = at[u] == pk0 + 4 * n ? g_n : (int)g[u];
        w[u] = row_imin((int)low[u], row_imax(gk, d));
    }
    if (!r.strict) {
        // the lowest split of a run of equal P whose g does not exceed the value (others cannot tie)
        const int *G = T - lane - 1;  // G[k] = g[k], k > n
        int a[2], v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            a[u] = row_imax(r.run[(at[u] - pk0) >> 2], n);
            v[u] = w[u] | r.kmask;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = (at[u] - pk0) >> 2;
            while (a[u] < j && (a[u] > n ? G[a[u]] : g_n) > v[u]) ++a[u];
            w[u] = a[u] < j ? (w[u] & ~r.kmask) | a[u] : w[u];
        }
    }
    row_lds_sync();
    w[0] = lane >= n ? w[0] : PP_INF32;
#pragma unroll
    for (int u = 0; u < 2; ++u) T[64 * u + 1] = w[u];
    return rounds;
}

template <int BANDS>
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

    constexpr int U = 2;  // two chunks of 64 cells
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int S = a.S, K = a.K, L = a.L, D = a.D;
    const int RS = dpr_stride(L);  // row stride: keys in dwords, arena rows in bytes
    const int kmask = (1 << K) - 1;
    const size_t lds_wave = dpr_lds_per_wave(L, S, a.rows, a.g.stages);
    // (P[k] << K) - k, k = 0..128 (P padded with P[L]), shared by the workgroup.  A search looks up to 64
    // entries below split 0: what stands there ends it.  It lies behind the waves' parts, because the search
    // looks as far below their rows.
    int *sPk = (int *)(smem + lds_wave * (blockDim.x >> 6)) + 64;
    for (int k = threadIdx.x; k < 64; k += blockDim.x) sPk[k - 64] = (int)0x80000001;
    for (int k = threadIdx.x; k <= 64 * U; k += blockDim.x) sPk[k] = (a.g.p32[k < L ? k : L] << K) - k;
    __syncthreads();
    unsigned char *run = (unsigned char *)(sPk + 64 * U + 1);
    for (int k = threadIdx.x; k < 64 * U; k += blockDim.x) {
        int a = k;
        while (a > 0 && sPk[a - 1] + (a - 1) == sPk[k] + k) --a;
        run[k] = (unsigned char)a;
    }
    __syncthreads();
    unsigned char *mine = smem + (size_t)wib * lds_wave;
    const int arena_rows = dpr_arena_rows(S, a.g.stages), key_rows = a.rows;
    int *rows = (int *)mine;                           // [key_rows][RS]: the current path's rows
    int *tops = rows + key_rows * RS + (128 - L);      // [pending][S] key of cell (n, L)
    unsigned char *arena = (unsigned char *)(tops + (a.g.stages ? DPR_PENDING * S : 0));
    unsigned char *slots = arena + (size_t)arena_rows * RS + (128 - L);  // [pending][S] arena row of row n
    const bool stages = a.g.stages != 0;
    const int tri = S * (S + 1) / 2;
    long long *C_out = a.g.C_out;
    int *bounds_out = a.g.bounds_out;
    const int *ord = a.g.ord;

    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + wib;
    const long long c0 = wave * a.chunk;
    const long long c1 = c0 + a.chunk < a.N ? c0 + a.chunk : a.N;

    // candidates of the chunk that bands have finished are passed by: pieces of it and what is left of them
    unsigned long long *reach, left;
    bool whole = band_begin<BANDS>(a, smem, reach, left);
    if (c0 >= c1) return;

    // row 0: one stage holding the first l layers (same for every candidate)
    for (int l = lane; l <= 64 * U; l += 64) rows[l] = sPk[l] + l;
    row_lds_sync();
    const int PLk = sPk[L] + L;
    rows_row r;
    r.rows = rows;
    r.PK = sPk;
    r.RS = RS;
    r.L = L;
    r.K = K;
    r.kmask = kmask;
    r.lane = lane;
    r.strict = row_is_strict(sPk, L, lane);
    r.run = run;
    int to_end[U];  // P[L] - P[l] of the lane's cells, infinite from L on
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = 64 * u + lane + 1;
        r.Pl[u] = (unsigned)(sPk[l] + l);
        r.last[u] = row_addr(sPk) + 4 * row_imin(l - 1, L - 1);
        to_end[u] = l < L ? PLk - sPk[l] : PP_INF32;
    }
    int v_steps = dpr_steps(L, lane);  // lane n: steps of a search in row n
    const unsigned long long smask = S >= 64 ? ~0ull : ((1ull << S) - 1);
    const int top_lane = (L - 1) & 63;  // the lane of cell L (in the last chunk)

    // up to DPR_PENDING finished candidates wait for their plans to be written out; lane q keeps the key
    // of cell (S-1, L) of the q-th of them (-1: its ordering was bad) and its place in the chunk (BAND_USE_NOT: they
    // are neighbours, pend0 the first)
    int pending = 0, v_top = 0, v_at = 0, pend0 = 0;
    unsigned long long pairs = 0, nrows = 0;  // work done by this wave
    int arena_used = 0;
    bool fresh = true;  // the arena was emptied: the next candidate must recompute every row
    int v_cur = 0;  // lane n: arena row holding the split indices of row n of the current path
    // lane n: key of cell (n, L) of the current path, i.e. the result for n+1 stages
    int v_tops = PLk;

    auto remember = [&](int top, int at) __attribute__((always_inline)) {
        if (lane == pending) {
            v_top = top;
            if (BANDS != BAND_USE_NOT) v_at = at;
        }
    };

    // Writes out C and the plans of all pending candidates, one per lane.
    auto flush = [&]() {
        row_lds_sync();
        const bool live = lane < pending;
        const long long cq = c0 + (BANDS == BAND_USE_NOT ? pend0 + lane : v_at);
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
            remember(bad ? -1 : key, (int)(c - c0));
            if (++pending == DPR_PENDING) flush();
        }
        if (pending) flush();
        return;
    }

    // Candidates by their place in the chunk: base .. end - 1 is the piece at hand.
    const int count = (int)(c1 - c0);
    const int piece = BANDS == BAND_USE_NOT ? count : (count + ((count + 63) >> 6) - 1) / ((count + 63) >> 6);
    int base = 0, end_c = count;
    bool whole_now = whole;
    auto next = [&](int c) -> int {
        if (BANDS == BAND_USE_NOT || whole_now) return c + 1;
        const unsigned long long m = left >> (c - base) >> 1;
        return m ? c + 1 + __builtin_ctzll(m) : end_c;
    };
    const int *ords = ord + c0 * S;

    // Lane n carries device o[n] of the candidate (v_o) and the link index o[n-1]*D + o[n]
    // that row n needs (v_link).
    int v_prev = 0;
    bool have_prev = false;
    int v_o = 0;

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
            const int k = 64 * u + lane + 1;
            x[u] = xp[k];  // (from L on: whatever follows the row in the workspace; not used)
        }
    };

    // prio_until[k]: the last candidate with more than prio_left[k] candidates still to do
    // (itself included)
    int prio_until[3];
    for (int k = 0; k < 3; ++k) prio_until[k] = count - 1 - a.prio_left[k];

    for (; base < count; base = end_c) {
    end_c = count;
    whole_now = whole;
    if (BANDS != BAND_USE_NOT && !whole) {
        end_c = band_piece<BANDS>(a, reach, c0, base, base + piece < count ? base + piece : count, left);
        if (!left) continue;
        whole = BANDS == BAND_USE_INSIDE && 2 * __builtin_popcountll(left) > end_c - base;
        have_prev = false;
        arena_used = 0;
        fresh = true;
    }
    // first candidate of the piece (bad ones are recorded and skipped)
    int c = BANDS == BAND_USE_NOT || whole_now ? base : base + __builtin_ctzll(left);
    v_o = lane < S ? ords[(long long)c * S + lane] : 0;
    int first = inspect(v_o);
    while (first < 0) {
        remember(-1, c);
        if (++pending == DPR_PENDING) flush();
        c = next(c);
        if (c >= end_c) break;
        v_o = lane < S ? ords[(long long)c * S + lane] : 0;
        first = inspect(v_o);
    }
    if (c >= end_c) {
        if (pending) flush();
        continue;
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
        int c_n = next(c);
        const bool more = c_n < end_c;
        int v_on = (more && lane < S) ? ords[(long long)c_n * S + lane] : 0;
        int first_n = -2, v_link_n = 0;  // next candidate: -2 none, -1 bad ordering
        bool flush_after = false;

        // candidate finished with key `top` in cell (S-1, L): remember it and the arena rows of
        // its path
        auto finish_candidate = [&](int top) __attribute__((always_inline)) {
            remember(top, c);
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
                } else {
                    flush_after = pending + 2 > DPR_PENDING;  // (and one that is bad needs a lane, too)
                }
            }
            fetch_x(xf, next_link);

            if (n < S - 1) {
                int w[U];
                const int steps = __builtin_amdgcn_readlane(v_steps, n);
                const int rounds = rows_compute(r, n, steps, xc, w);
                pairs += (unsigned long long)((L - n) * (rounds * steps + 1));
                ++nrows;
                if (rounds > 1 && lane == n && v_steps < key_rows - n && v_steps < DPR_MAX_STEPS) ++v_steps;
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
                        m = row_imin(m, row_imax(row_imax(wk, xk2), to_end[u]));
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
                    const int k = 64 * u + lane + 1;
                    const int xk2 = (int)((unsigned)xc[u] << K) | k, wk = (rows[(n - 1) * RS + k] & ~kmask) | k;
                    const int t = row_imax(row_imax(wk, xk2), to_end[u]);
                    m = k >= n ? row_imin(m, t) : m;
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
            remember(-1, c_n);
            if (++pending == DPR_PENDING) flush();
            c_n = next(c_n);
            first_n = -2;
            if (c_n < end_c) {
                v_on = lane < S ? ords[(long long)c_n * S + lane] : 0;
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
        c = c_n;
        v_o = v_on;
        v_link = v_link_n;
        first = first_n;
    }
    if (pending) flush();
    }
    if (lane == 0) pp_count_work(a.g.hdr, pairs, nrows, (unsigned)wave);
}

static size_t rows_own_lds(int L, int S, int rows, int stages, int wpb) {
    return (DPR_TABLE + (size_t)wpb * dpr_lds_per_wave(L, S, rows, stages) + 15) & ~(size_t)15;
}
static size_t rows_lds(int L, int D, int S, int rows, int stages, int wpb) {
    size_t lds = rows_own_lds(L, S, rows, stages, wpb);
    const size_t generic = dp_generic_lds_bytes(L);  // the int64 fallback's rows
    if (lds < generic) lds = generic;
    const size_t flat = pp_flat_lds_wanted(L, D, S, wpb);  // the closed-form body's tables
    return lds < flat ? flat : lds;
}

dpr_shape pp_dp_rows_shape(int L, int D, int S, int stages) {
    dpr_shape s = {4, dpr_min_rows(L, S), 1, 0};
    while (s.wpb && rows_lds(L, D, S, s.rows, stages, s.wpb) > 64 * 1024) s.wpb >>= 1;
    if (!s.wpb) return s;
    // workgroups on a compute unit: 160 KiB of LDS, given out in pieces of 1280 bytes
    auto groups = [&](int rows) {
        const size_t lds = rows_lds(L, D, S, rows, stages, s.wpb);
        return lds > 64 * 1024 ? 0 : (int)(160 * 1024 / ((lds + 1279) / 1280 * 1280));
    };
    const int g = groups(s.rows);
    while (S > 2 && s.rows < S - 2 + DPR_MAX_STEPS && groups(s.rows + 1) == g) ++s.rows;
    s.lds = rows_lds(L, D, S, s.rows, stages, s.wpb);
    s.waves_per_cu = g * s.wpb > 16 ? 16 : g * s.wpb;
    return s;
}

int pp_launch_dp_rows(const dp_rows_args &a, int grid, const dpr_shape &sh, hipStream_t st) {
    dp_rows_args b = a;
    b.rows = sh.rows;
    const int use = !a.g.band ? BAND_USE_NOT : a.g.left ? BAND_USE_ALONE : BAND_USE_INSIDE;
    size_t lds = sh.lds;
    b.links_at = b.pooled = 0;
    if (use == BAND_USE_INSIDE) {
        // the words of the links: in the waves' place, or behind it where that costs no workgroup
        const size_t own = rows_own_lds(a.L, a.S, sh.rows, a.g.stages, sh.wpb), words = band_link_bytes(a.D, a.S, a.g.stages);
        b.pooled = a.chunk < 64 && words && words <= sh.wpb * dpr_lds_per_wave(a.L, a.S, sh.rows, a.g.stages);
        const size_t to = own + words > lds ? own + words : lds;
        auto groups = [&](size_t bytes) { return (int)(160 * 1024 / ((bytes + 1279) / 1280 * 1280)); };
        if (!b.pooled && words && to <= 64 * 1024 && (groups(to) >= groups(lds) || groups(to) * sh.wpb >= 16)) {
            b.links_at = (int)own;
            lds = to;
        }
    }
    b.g.lds_bytes = lds;
    if (use == BAND_USE_ALONE) hipLaunchKernelGGL(k_dp_rows<BAND_USE_ALONE>, dim3(grid), dim3(64 * sh.wpb), lds, st, b);
    else if (use == BAND_USE_INSIDE) hipLaunchKernelGGL(k_dp_rows<BAND_USE_INSIDE>, dim3(grid), dim3(64 * sh.wpb), lds, st, b);
    else hipLaunchKernelGGL(k_dp_rows<BAND_USE_NOT>, dim3(grid), dim3(64 * sh.wpb), lds, st, b);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
