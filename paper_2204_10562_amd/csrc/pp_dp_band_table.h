// The table of the bands (pp_dp_band.h), built by one workgroup of the pack kernel.
//
// What bounds it: the latency of chains through LDS, one step per stage (where the next cut can be, in two reads:
// a bucket of the prefix sums, then four entries of them), 64 times side by side; then the channel-free program
// over the bands' cells, a row per stage.  8 stages 9 us where the pack kernel took 7.5 without it, 16 stages 12 us,
// 32 24 us.
#pragma once

#include "pp_dp_band.h"

struct band_table_args {
    int L, D, S, K;
    const long long *PF, *PB, *XF, *XB;
    int *table;                    // NULL: not wanted
    int waves;                     // waves that find the bands
    int stages;
    int cells;                     // the recursion over the bands' cells is worth trying: 0 no, 1 if links allow, 2 yes
    unsigned long long fit_limit;  // of the 32-bit keys
};

// Of so many transfer times all over the table, the part that is longer than a stage says what bands are good for.
// A candidate has the channel-free plan if none of its S - 1 cuts has one: not likely where they are more than a
// (S - 1)th.  The recursion moves cuts to where there is none, p / (1 - p) cells away on an average, and all of its
// cuts together have about a band to move in.
#define BAND_SAMPLE 2  // per thread

// The bands of pp_dp_band.h.  P: the prefix sums in LDS, with 0 before them
// and a large number twice behind; inv[b]: the first k with
// P[k] >= b << sh.
struct band_model {
    const int *P;
    const unsigned short *inv;
    int L, sh, longest, total;
    // the number of k with P[k] <= t, 0 <= t < P[L]; p: the last of those P[k].  (Four entries at once: a
    // bucket seldom holds more, and a chain of such steps is what the whole block takes.)
    __device__ __forceinline__ int upto(int t, int &p) const {
        int k = inv[t >> sh];
        const int p0 = P[k - 1], p1 = P[k], p2 = P[k + 1], p3 = P[k + 2];
        p = p1 <= t ? (p2 <= t ? p2 : p1) : p0;
        k += (p1 <= t) + (p2 <= t);
        if (p3 <= t) {
            p = p3;
            while (P[++k] <= t) p = P[k];
        }
        return k;
    }
    // how far stage n gets from cell l (P[l] = p), at most v long, if every stage after it keeps a layer
    __device__ __forceinline__ void forth(int &l, int &p, int n, int xi, int v) const {
        const int most = L - (xi - 1 - n), t = p + v;
        l = upto(band_min(t, total - 1), p) - 1;
        if (l > most || t >= total) { l = most; p = P[l]; }
    }
    // the first cell of row n from which a stage of at most v reaches cell l of row n + 1 (P[l] = p)
    __device__ __forceinline__ void back(int &l, int &p, int n, int v) const {
        const int t = p - v - 1;
        l = band_max(t < 0 ? 0 : upto(t, p), n + 1);
        p = P[l];
    }
};

// One wave, a time per lane: how far xi stages of at most v get from the left (hi, rows of 64 columns) and from
// the right (lo), and the most cells of a band.  Returns whether the layers fit.
__device__ __forceinline__ bool band_reach(const band_model &m, int xi, int v, unsigned short *hi, unsigned short *lo, int &most) {
    const int lane = threadIdx.x & 63;
    int l = 0, p = 0, r = m.L, q = m.total;
    for (int n = 0; n + 1 < xi; ++n) {
        m.forth(l, p, n, xi, v);
        m.back(r, q, xi - 2 - n, v);
        hi[n * 64 + lane] = (unsigned short)l;
        lo[(xi - 2 - n) * 64 + lane] = (unsigned short)r;
    }
    hi[(xi - 1) * 64 + lane] = lo[(xi - 1) * 64 + lane] = (unsigned short)m.L;
    most = 1;
    for (int n = 0; n + 1 < xi; ++n) most = band_max(most, hi[n * 64 + lane] - lo[n * 64 + lane] + 1);
    return p + v >= m.total;
}

// Writes a level's bands from column `lane_of` of hi and lo (v = 0: there are none).
__device__ __forceinline__ void band_write(const band_table_args &a, int xi, int level, int v, int lane_of, const unsigned short *hi,
                                           const unsigned short *lo) {
    const int lane = threadIdx.x & 63;
    if (lane == 0) a.table[band_top_at(a.S, level, xi)] = v ? (v << a.K) | ((1 << a.K) - 1) : -1;
    if (!v) return;
    int *rows = a.table + band_row_at(a.S, level, xi);
    for (int n = lane; n < xi; n += 64) rows[n] = lo[n * 64 + lane_of] | (hi[n * 64 + lane_of] - lo[n * 64 + lane_of] + 1) << 16;
}

// The times a lane tries: for level 0 `n` times from the average stage (or the longest layer) on, of which the
// last is enough, because a stage longer than v - longest cannot take another layer; for level 1 up to about five
// times that.
__device__ __forceinline__ int band_time(const band_model &m, int xi, bool wide, int i, int n) {
    const int v0 = band_max(m.longest, (int)(((long long)m.total + xi - 1) / xi));
    const long long v = wide ? v0 + (long long)v0 * i * i / (n * n / 4) : v0 + (long long)i * ((m.longest + n - 2) / (n - 1));
    return v < m.total ? (int)v : m.total;
}

// Level 1, from what band_reach has left in the columns first .. first + n - 1: the largest time whose bands have
// at most BAND_CELLS cells, if the layers fit.  (Times that are too short have empty bands.)
__device__ __forceinline__ void band_wide(const band_table_args &a, int xi, int mine, bool fits, int most, unsigned long long lanes,
                                          const unsigned short *hi, const unsigned short *lo) {
    const unsigned long long good = __ballot(fits && most <= BAND_CELLS) & lanes;
    const int col = good ? 63 - __builtin_clzll(good) : 0;
    band_write(a, xi, 1, good ? band_max(1, __builtin_amdgcn_readlane(mine, col)) : 0, col, hi, lo);
}

// Level 0: the smallest time with which the layers fit, and what the channel-free program does in its bands.
__device__ inline void band_tight(const band_table_args &a, const band_model &m, int xi, int mine, bool fit, int most, unsigned long long lanes,
                           unsigned short *hi, unsigned short *lo) {
    const int lane = threadIdx.x & 63, S = a.S, L = a.L, K = a.K, kmask = (1 << K) - 1, *P = m.P;
    const unsigned long long fits = __ballot(fit) & lanes;
    const int col = fits ? __builtin_ctzll(fits) : 0;
    const bool there = fits && __builtin_amdgcn_readlane(most, col) <= BAND_CELLS;
    int *C = a.table + band_C_at(S, xi), *plan = a.table + band_plan_at(S, xi);
    band_write(a, xi, 0, there ? band_max(1, __builtin_amdgcn_readlane(mine, col)) : 0, col, hi, lo);
    if (!there) {
        if (lane == 0) *C = -1;
        return;
    }
    // lane n of v_lo, v_w: row n; lane i of the others: cell i of the band
    const int v_lo = lane < xi ? lo[lane * 64 + col] : L, v_w = lane < xi ? hi[lane * 64 + col] - v_lo + 1 : 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int lo_p = __builtin_amdgcn_readlane(v_lo, 0), w_p = __builtin_amdgcn_readlane(v_w, 0);
    int p_p = P[band_min(lo_p + lane, L)], W = p_p << K;
    int lo_n = __builtin_amdgcn_readlane(v_lo, 1), w_n = __builtin_amdgcn_readlane(v_w, 1), p_n = P[band_min(lo_n + lane, L)];
    for (int n = 1; n < xi; ++n) {
        const int after = n + 1 < xi ? n + 1 : n;
        const int lo_a = __builtin_amdgcn_readlane(v_lo, after), w_a = __builtin_amdgcn_readlane(v_w, after);
        const int p_a = P[band_min(lo_a + lane, L)];  // (a row ahead: the chain is W's alone)
        const int cell = lo_n + lane, split = lo_p + lane;
        int best = PP_INF32;
        for (int k = 0; k < w_p; ++k) {
            const int at = lo_p + k, g = (__builtin_amdgcn_readlane(W, k) & ~kmask) | at;
            const int p_at = __builtin_amdgcn_readlane(p_p, k);
            const int d = at < cell ? ((p_n - p_at) << K) | at : PP_INF32;
            best = band_min(best, band_max(g, d));
        }
        // the longest time of a link at this lane's split that changes no cell
        const int next = band_max(lo_n, split + 1);
        const int p_next = P[band_min(next, L)];
        if (lane < w_p)
            a.table[band_hidden_at(S, xi, n) + lane] = next < lo_n + w_n ? band_max(W >> K, p_next - p_p) : PP_INF32;
        if (lane < w_n) hi[n * 64 + lane] = (unsigned short)(best & kmask);  // (the cell's split)
        W = best;
        lo_p = lo_n; w_p = w_n; p_p = p_n;
        lo_n = lo_a; w_n = w_a; p_n = p_a;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // (all lanes follow the chain; lane n keeps bound n)
    int e = L, v_e = L;
    for (int n = xi - 1; n >= 1; --n) {
        if (lane == n) v_e = e;
        e = __builtin_amdgcn_readfirstlane(hi[n * 64 + e - __builtin_amdgcn_readlane(v_lo, n)]);
    }
    if (lane == 0) { v_e = e; *C = W >> K; }
    if (lane < xi) plan[lane] = v_e;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Buckets of the table that finds a prefix sum: a power of two, about eight per layer.
__host__ __device__ static inline int band_buckets(int L) {
    int nb = 64;
    while (nb < 8 * L && nb < 8192) nb <<= 1;
    return nb;
}
// LDS of the block that finds the bands: the prefix sums, the buckets, and 2 S rows of 64 columns per wave (one
// wave per level; the search over stage counts: as many as fit, a count at a time each).
static inline size_t band_table_lds(int L, int S, int stages, int &waves) {
    const size_t model = (((size_t)(L + 12) * 4 + 15) & ~(size_t)15) + (size_t)band_buckets(L) * 2;
    waves = stages ? 4 : 2;
    while (stages && waves > 1 && model + (size_t)waves * S * 256 > 63 * 1024) waves >>= 1;
    return model + (size_t)waves * S * 256;
}

__device__ inline void band_table(const band_table_args &a, unsigned char *sh) {
    const int L = a.L, S = a.S, tid = threadIdx.x;
    int *s_longest = (int *)sh, *s_differs = s_longest + 4, *s_sample = s_longest + 5, *P = s_longest + 9;
    unsigned short *inv = (unsigned short *)(sh + (((size_t)(L + 12) * 4 + 15) & ~(size_t)15));
    const int nb = band_buckets(L);
    unsigned short *reach = inv + nb;
    const long long total = a.PF[L] + a.PB[L];
    // Where no link's time differs between the first two cut positions it probably differs nowhere, and the
    // closed form needs no bands.  (Requested together with the prefix sums.)
    bool differs = L < 3 || a.D > 64;
    for (int link = tid; !differs && link < a.D * a.D; link += 256) {
        const size_t at = (size_t)link * L;
        differs = a.XF[at] + a.XB[at] != a.XF[at + 1] + a.XB[at + 1];
    }
    bool fits = total > 0 && (unsigned long long)total < a.fit_limit;
    int longest = 0;
    for (int l = tid; l <= L; l += 256) {
        const long long p = a.PF[l] + a.PB[l], q = l ? a.PF[l - 1] + a.PB[l - 1] : 0;
        P[l] = (int)p;
        fits &= p >= q && p <= total;
        longest = band_max(longest, (int)(p - q));
    }
    // (requested here, looked at when the buckets are there)
    long long sample[BAND_SAMPLE];
    if (a.cells < 2) {
#pragma unroll
        for (int j = 0; j < BAND_SAMPLE; ++j) {
            const unsigned at = (unsigned)(tid * BAND_SAMPLE + j) * 2654435761u;  // (spread over links and cuts)
            const int link = (int)((at >> 16) * (unsigned)(a.D * a.D) >> 16), k = (int)((at & 0xffff) * (unsigned)(L - 1) >> 16);
            const size_t i = (size_t)link * L + k;
            sample[j] = a.XF[i] + a.XB[i];
            if (link % (a.D + 1) == 0) sample[j] = -1;  // (a device and itself)
        }
    }
    for (int off = 32; off; off >>= 1) longest = band_max(longest, __shfl_xor(longest, off));
    if ((tid & 63) == 0) s_longest[tid >> 6] = longest;
    if (tid == 0) *s_differs = s_sample[0] = s_sample[1] = 0;
    __syncthreads();
    longest = band_max(band_max(s_longest[0], s_longest[1]), band_max(s_longest[2], s_longest[3]));
    if (differs) *s_differs = 1;
    auto none = [&]() {
        for (int i = tid; i < BAND_LEVELS * S; i += 256) a.table[i] = -1;
        for (int i = tid; i < S; i += 256) a.table[band_C_at(S, i + 1)] = -1;
    };
    if (!__syncthreads_and(fits) || !*s_differs) return none();
    band_model m;
    m.P = P;
    m.inv = inv;
    m.L = L;
    m.longest = longest;
    m.total = P[L];
    m.sh = 0;
    while (P[L] >> m.sh >= nb) ++m.sh;
    if (tid == 0) { P[-1] = 0; P[L + 1] = P[L + 2] = PP_INF32; }
    // (bucket b begins with the first layer that ends at b << sh or later)
    for (int k = tid; k <= L; k += 256) {
        const int from = k ? (P[k - 1] >> m.sh) + 1 : 0, to = P[k] >> m.sh;
        for (int b = from; b <= to; ++b) inv[b] = (unsigned short)k;
    }
    if (a.cells < 2) {
        int seen = 0, over = 0;
#pragma unroll
        for (int j = 0; j < BAND_SAMPLE; ++j) {
            seen += __builtin_popcountll(__ballot(sample[j] >= 0));
            over += __builtin_popcountll(__ballot(sample[j] > longest && sample[j] > total / S));
        }
        if ((tid & 63) == 0) { atomicAdd(&s_sample[0], seen); atomicAdd(&s_sample[1], over); }
    }
    __syncthreads();
    if (s_sample[1] * (S - 1) > (a.cells ? 3 * BAND_CELLS / 4 * (s_sample[0] - s_sample[1]) : s_sample[0])) return none();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave >= a.waves) return;
    unsigned short *hi = reach + (size_t)wave * 2 * S * 64, *lo = hi + (size_t)S * 64;
    const int lane = tid & 63;
    int most;
    if (a.stages) {
        // (one stage: nothing to cut)
        if (tid == 0) { a.table[band_plan_at(S, 1)] = L; a.table[band_C_at(S, 1)] = P[L]; }
        for (int xi = S - wave; xi >= 2; xi -= a.waves) {
            // (half of the lanes for each level)
            const int mine = band_time(m, xi, lane >= 32, lane & 31, 32);
            const bool fits = band_reach(m, xi, mine, hi, lo, most);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            band_wide(a, xi, mine, fits, most, ~0ull << 32, hi, lo);
            band_tight(a, m, xi, mine, fits, most, ~0ull >> 32, hi, lo);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    } else {
        const int mine = band_time(m, S, wave != 0, lane, 64);
        const bool fits = band_reach(m, S, mine, hi, lo, most);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (wave) band_wide(a, S, mine, fits, most, ~0ull, hi, lo);
        else band_tight(a, m, S, mine, fits, most, ~0ull, hi, lo);
    }
}
