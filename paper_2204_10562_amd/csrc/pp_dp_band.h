// A candidate's partition from the few cells of every row that a good plan can use, one lane per candidate.
//
// Recursion for W(l, xi, r, i) of Sec. IV-B / the PRM listing with one replica per stage:
//   W[n][l] = min_{n<=k<l} max(W[n-1][k], X_n[k], P[l] - P[k]),   C = W[S-1][L],
// lowest minimising k kept.  Let v be any time, and band n the cells lo_n .. hi_n of row n: hi_n is as far as
// n + 1 stages of at most v get from the left when transfers are free, lo_n as far as the S - 1 - n others get
// from the right.  A cell (n, l) of a band with W[n][l] <= v has all splits k that attain its value in band
// n - 1: W[n-1][k] <= v, and the value with transfers is no smaller than without, so k <= hi_{n-1}; and
// P[l] - P[k] <= v, so from k the rest still fits, k >= lo_{n-1}.  The recursion over the bands' cells alone
// therefore has, by induction, the true value and the true lowest split wherever the value is at most v, and a
// value above v elsewhere.  If it ends at or below v, C and the plan are the exact ones; otherwise the
// candidate is left to the kernels that compute whole rows.
//
// The bands do not depend on the candidate, so the pack kernel finds them once: at the smallest v with which
// the model can be cut at all (to 1/63 of the longest layer, or 1/31), and at the largest for which no band is
// wider than BAND_CELLS.  Where transfers seldom take longer than a stage, which is what a pipeline is for,
// nearly all candidates end at the first: its bands hold 1 to 4 cells of a row's hundreds.  Those whose links
// bind need the second or whole rows.  And a link whose times are hidden behind the other two terms in every cell
// of its row's band changes nothing: a candidate of such links alone has the plan of the channel-free program,
// which is one for all of them (band_free_try).
//
// 2^20 candidates of L = 1024, S = 32, the partition alone: 97.7 ms with whole rows, 0.21 ms (0.76 ms with the
// recursion over the bands' cells for each); 20 011 of L = 400, S = 48 1.54 ms -> 23 us; 15 751 of L = 300, S = 16
// 212 -> 13 us; all 8! orderings of L = 128 48 -> 15 us; 200 003 of L = 97, S = 11 894 -> 35 us.
#pragma once

#include "pp_common.h"
#include "pp_dp_generic.h"

#define BAND_CELLS 16  // most cells of a band
#define BAND_LEVELS 2
// Whether and where they are tried (pp_dp.hip, band_use).
enum { BAND_USE_NOT, BAND_USE_INSIDE, BAND_USE_ALONE };

// The table the pack kernel leaves (ints): per level the key up to which stage count xi = 1..S ends well (-1:
// there is no such band), then per level lo | cells << 16 of row n of xi stages at xi (xi - 1) / 2 + n.
__host__ __device__ static inline int band_top_at(int S, int level, int xi) { return level * S + xi - 1; }
__host__ __device__ static inline int band_row_at(int S, int level, int xi) {
    return BAND_LEVELS * S + level * (S * (S + 1) / 2) + xi * (xi - 1) / 2;
}

// Then what the channel-free program does in the first level's bands (plans of S stages only, or of every stage
// count): its bounds in the places of the rows, its C per stage count (-1: there is none), and BAND_CELLS times
// per row n >= 1: the longest time of row n's link at each split of band n - 1 that is hidden behind the other
// two terms in every cell of band n.
__host__ __device__ static inline int band_plan_at(int S, int xi) { return band_row_at(S, BAND_LEVELS, xi); }
__host__ __device__ static inline int band_C_at(int S, int xi) { return band_row_at(S, BAND_LEVELS + 1, 1) + xi - 1; }
__host__ __device__ static inline int band_hidden_at(int S, int xi, int n) {
    return band_C_at(S, S + 1) + (xi * (xi - 1) / 2 + n) * BAND_CELLS;
}

// Lists of at least dp_args::band_all candidates are looked at with the recursion over the bands' cells, shorter ones
// for the channel-free plan alone.

// LDS of one wave: a column of splits (4 bits a cell) and one of devices per lane.  Lists of fewer than a wave's
// candidates are left to the other kernels (pp_band_wanted).
__host__ __device__ static inline size_t band_lds_per_wave(int S) {
    return (size_t)S * 64 * 4 * (BAND_CELLS / 8) + (size_t)S * 64;
}

struct band_int4 { int v[4]; };  // (16 bytes in one load, aligned to 4)

__device__ __forceinline__ int band_max(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ int band_min(int a, int b) { return a < b ? a : b; }

// Whether row n's link reaches into a value of the plan with xi stages.
__device__ __forceinline__ bool band_link_reaches(const dp_args &a, const int *table, int xi, int link, int n) {
    const int band = table[band_row_at(a.S, 0, xi) + n - 1], lo = band & 0xffff, w = band >> 16;
    const int *x = a.x32 + (size_t)link * a.L + lo, *most = table + band_hidden_at(a.S, xi, n);
    bool reaches = false;
    for (int k = 0; k < w; ++k) reaches |= x[k] > most[k];
    return reaches;
}

// Which links reach into which rows: for plans of S stages a word per link with a bit per row, for plans of
// every stage count a word per row (from row 1 on) and link with a bit per count.
__host__ __device__ static inline int band_link_words(int D, int S, int stages) { return D * D * (stages ? S - 1 : 1); }
// The words built by a workgroup for itself: where that is a few reads per thread.
#define BAND_LINK_WORDS 512
#define BAND_LINK_ROWS 4096
__host__ __device__ static inline size_t band_link_bytes(int D, int S, int stages) {
    if (S < 2 || D > 32 || band_link_words(D, S, stages) > BAND_LINK_WORDS) return 0;
    if (D * D * (stages ? S * (S - 1) / 2 : S - 1) > BAND_LINK_ROWS) return 0;
    return (size_t)band_link_words(D, S, stages) * 8 + 32;  // (and a word per wave in front)
}
__device__ __forceinline__ void band_links(const dp_args &a, const int *table, unsigned long long *links) {
    const int S = a.S, nl = a.D * a.D, words = band_link_words(a.D, S, a.stages);
    if (!a.stages) {
        for (int i = threadIdx.x; i < words; i += blockDim.x) links[i] = 0;
        __syncthreads();
    }
    for (int i = threadIdx.x; i < (S - 1) * nl; i += blockDim.x) {
        const int n = i / nl + 1, link = i - (n - 1) * nl;
        if (a.stages) {
            unsigned long long m = 0;
            for (int xi = n + 1; xi <= S; ++xi)
                if (band_link_reaches(a, table, xi, link, n)) m |= 1ull << (xi - 1);
            links[i] = m;
        } else if (band_link_reaches(a, table, S, link, n)) {
            // (a row of a link per thread: with a link per thread it is a chain of S trips to memory)
            atomicOr(&links[link], 1ull << n);
        }
    }
}

// Whether there are channel-free plans of all the stage counts asked for.
__device__ __forceinline__ bool band_free(const dp_args &a, const int *table) {
    const int lane = threadIdx.x & 63;
    const bool none = lane < a.S && (a.stages || lane == a.S - 1) && table[band_C_at(a.S, lane + 1)] < 0;
    return !__ballot(none);
}

// A wave's candidates, one per lane (c, where live; all lanes must call): reports bad orderings, and finishes the
// candidates none of whose links reaches into its row (links: band_links' words, or NULL: there are none) with
// the channel-free plan.  Returns the others, a bit per lane.
__device__ __forceinline__ unsigned long long band_free_try(const dp_args &a, const int *table, const unsigned long long *links,
                                                            long long c, bool live) {
    const int lane = threadIdx.x & 63, S = a.S, D = a.D, tri = S * (S + 1) / 2;
    const int *row = a.ord + c * S;
    bool bad = false;
    unsigned long long seen = 0, reach = 0;
    int before = 0, first = lane ? S : 0;  // the first place where the devices differ from those of the lane before
    auto device = [&](int n, int d) {
        const int left = __builtin_amdgcn_update_dpp(d, d, DPP_WAVE_SHR1, 0xf, 0xf, false);
        if (d != left && first == S) first = n;
        if (a.validate) {
            bad |= d < 0 || d >= D;
            d = bad ? 0 : d;
            bad |= (seen >> d) & 1;
            seen |= 1ull << d;
        }
        if (links && n) reach |= a.stages ? links[((n - 1) * D + before) * D + d] : links[before * D + d] & 1ull << n;
        before = d;
    };
    if ((S & 3) == 0 && ((uintptr_t)a.ord & 15) == 0) {
        for (int n = 0; n < S; n += 4) {
            const int4 v = live ? *(const int4 *)(row + n) : make_int4(0, 1, 2, 3);
            device(n, v.x); device(n + 1, v.y); device(n + 2, v.z); device(n + 3, v.w);
        }
    } else {
        for (int n = 0; n < S; ++n) device(n, live ? row[n] : 0);
    }
    bad = bad && live;
    const int nb = a.stages ? tri : S, nc = a.stages ? S : 1;
    long long *Co = a.C_out + c * nc;
    int *bo = a.bounds_out + c * nb;
    if (bad) {
        pp_raise(a.status, PP_FAULT_ORDERING);
        for (int n = 0; n < nc; ++n) Co[n] = PP_INF64;
        for (int n = 0; n < nb; ++n) bo[n] = 0;
    }
    if (!links) return __ballot(live && !bad);
    const bool done = live && !bad && !reach;
    const unsigned long long ended = __ballot(done);
    if (!ended) return __ballot(live && !bad);
    // (a row of bounds is the table's)
    const int *plan = table + band_plan_at(S, a.stages ? 1 : S), *C = table + band_C_at(S, a.stages ? 1 : S);
    const bool vec4 = (nb & 3) == 0 && ((uintptr_t)a.bounds_out & 15) == 0;
    for (int n0 = 0; n0 < nb; n0 += 64) {
        const int v_plan = n0 + lane < nb ? plan[n0 + lane] : 0, end = nb - n0 < 64 ? nb - n0 : 64;
        if (vec4) {
            for (int n = 0; n < end; n += 4) {
                const int4 v = make_int4(__builtin_amdgcn_readlane(v_plan, n), __builtin_amdgcn_readlane(v_plan, n + 1),
                                         __builtin_amdgcn_readlane(v_plan, n + 2), __builtin_amdgcn_readlane(v_plan, n + 3));
                if (done) *(int4 *)(bo + n0 + n) = v;
            }
        } else {
            for (int n = 0; n < end; ++n) {
                const int e = __builtin_amdgcn_readlane(v_plan, n);
                if (done) bo[n0 + n] = e;
            }
        }
    }
    const int v_C = lane < nc ? C[lane] : 0;
    for (int n = 0; n < nc; ++n) {
        const int e = __builtin_amdgcn_readlane(v_C, n);
        if (done) Co[n] = e;
    }
    // (rows of neighbours in the wave that begin with the same devices count once, the last row for everyone)
    const bool after = lane && (ended >> (lane - 1) & 1);
    int rows = done ? 1 + band_max(0, S - 1 - (after && first > 1 ? first : 1)) : 0;
    for (int off = 32; off; off >>= 1) rows += __shfl_xor(rows, off);
    if (lane == 0) {
        auto &w = a.hdr->work[(c >> 6) & 63];
        atomicAdd(&w.rows, (unsigned long long)rows);
        atomicAdd(&w.free_rows, (unsigned long long)rows);
    }
    return __ballot(live && !bad && !done);
}

// One link's words, by one wave; with a.fx also its times at the channel-free plan's cuts, the sign bit of the first saying that
// the link reaches into the row.
__device__ __forceinline__ void band_link_wave(const dp_args &a, const int *table, int link, unsigned long long *links) {
    const int lane = threadIdx.x & 63, S = a.S;
    if (S < 2 || !band_free(a, table)) return;
    if (!a.stages) {
        const unsigned long long rows = __ballot(lane >= 1 && lane < S && band_link_reaches(a, table, S, link, lane));
        if (lane == 0) links[link] = rows;
        if (a.fx && lane >= 1 && lane < S) {
            const size_t at = (size_t)link * a.L + (table[band_plan_at(S, S) + lane - 1] - 1);
            a.fx[(size_t)lane * a.D * a.D + link] = make_int2((int)a.XF[at] | (rows >> lane & 1 ? (int)0x80000000 : 0), (int)a.XB[at]);
        }
    } else if (lane >= 1 && lane < S) {
        unsigned long long m = 0;
        for (int xi = lane + 1; xi <= S; ++xi)
            if (band_link_reaches(a, table, xi, link, lane)) m |= 1ull << (xi - 1);
        links[(size_t)(lane - 1) * a.D * a.D + link] = m;
    }
}

// Groups of candidates a wave takes without a level, after one in which the level was of use to less than one
// in eight.
struct band_pace { int skip[BAND_LEVELS]; };

// The same with the bands: the candidates that no link's words finish go through the recursion over the cells of
// the first level's bands, and those it does not end for through the second's.  PK: (P[k] << K) - k for k = 0..L
// and BAND_CELLS more entries, in LDS; lds: band_lds_per_wave bytes, 16-byte aligned.  D <= 64.
__device__ __forceinline__ unsigned long long band_try(const dp_args &a, const int *table, const unsigned long long *links,
                                                       const int *PK, unsigned char *lds, long long c, bool live,
                                                       band_pace &pace) {
    constexpr int CELLS = BAND_CELLS, WORDS = CELLS / 8;
    const int lane = threadIdx.x & 63, S = a.S, L = a.L, D = a.D, K = a.K, kmask = (1 << K) - 1;
    unsigned *args = (unsigned *)lds + lane;                                       // [S][WORDS][64]
    unsigned char *dev = lds + (size_t)S * WORDS * 256 + lane;                      // [S][64]
    const unsigned long long most = band_free_try(a, table, links, c, live);
    if (!most) return 0;
    bool open = most >> lane & 1;  // this lane's candidate has ended well so far
    for (int n = 0; n < S; ++n) dev[n * 64] = open ? (unsigned char)a.ord[c * S + n] : 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int tri = S * (S + 1) / 2;
    unsigned long long pairs = 0;  // of all the lanes' bands
    int tried[BAND_LEVELS] = {}, well[BAND_LEVELS] = {};

    for (int xi = a.stages ? 1 : S; xi <= S; ++xi) {
        if (xi == 1) {
            if (open) {
                a.C_out[c * (a.stages ? S : 1)] = (PK[L] + L) >> K;
                a.bounds_out[c * (a.stages ? tri : S)] = L;
            }
            continue;
        }
        bool todo = open;
        for (int level = 0; level < BAND_LEVELS && __ballot(todo); ++level) {
            const int top_most = __builtin_amdgcn_readfirstlane(table[band_top_at(S, level, xi)]);
            if (pace.skip[level] > 0 || top_most < 0 || (level && top_most <= table[band_top_at(S, 0, xi)])) continue;
            const int v_row = lane < xi ? table[band_row_at(S, level, xi) + lane] : 0;
            int prev = __builtin_amdgcn_readlane(v_row, 0);
            int lo_p = prev & 0xffff, w_p = prev >> 16;
            int v_pp = PK[lo_p + (lane & (CELLS - 1))];
            int W[CELLS], x[CELLS];
#pragma unroll
            for (int k = 0; k < CELLS; ++k) W[k] = __builtin_amdgcn_readlane(v_pp, k) + lo_p + k;
            // the times of row n's link at the splits of band n - 1, four at a time
            auto fetch = [&](int n, int lo, int w) {
                const int *xp = a.x32 + ((size_t)dev[(n - 1) * 64] * D + dev[n * 64]) * L + lo;
#pragma unroll
                for (int k = 0; k < CELLS; k += 4)
                    if (k < w) {
                        const band_int4 v = *(const band_int4 *)(xp + k);
#pragma unroll
                        for (int u = 0; u < 4; ++u) x[k + u] = v.v[u];
                    }
            };
            fetch(1, lo_p, w_p);
            bool alive = todo;
            for (int n = 1; n < xi; ++n) {
                const unsigned long long here_too = __ballot(alive);
                if (!here_too) break;
                const int here = __builtin_amdgcn_readlane(v_row, n);
                const int lo = here & 0xffff, w = here >> 16;
                const int v_pn = PK[lo + (lane & (CELLS - 1))];
                int g[CELLS], pk[CELLS];
#pragma unroll
                for (int k = 0; k < CELLS; ++k) {
                    if ((k & ~3) >= w_p) continue;
                    const int at = lo_p + k;
                    const int gk = band_max((W[k] & ~kmask) | at, (int)((unsigned)x[k] << K) | at);
                    g[k] = k < w_p ? gk : PP_INF32;
                    pk[k] = __builtin_amdgcn_readlane(v_pp, k);
                }
                if (n + 1 < xi) fetch(n + 1, lo, w);
                int least = PP_INF32;
                unsigned word[WORDS];
#pragma unroll
                for (int q = 0; q < WORDS; ++q) word[q] = 0;
#pragma unroll
                for (int i = 0; i < CELLS; ++i) {
                    if (i >= w) continue;
                    const int l = lo + i, pl = __builtin_amdgcn_readlane(v_pn, i) + l;
                    int best = PP_INF32;
#pragma unroll
                    for (int k = 0; k < CELLS; ++k) {
                        if ((k & ~3) >= w_p) continue;
                        // (the same in all lanes; the splits of a group of four that are all too far away)
                        if (pl - pk[k | 3] > top_most && (k | 3) < w_p) continue;
                        const int d = lo_p + k < l ? pl - pk[k] : PP_INF32;
                        best = band_min(best, band_max(g[k], d));
                    }
                    least = band_min(least, best);
                    W[i] = best;
                    word[i / 8] |= ((unsigned)((best & kmask) - lo_p) & 15u) << (4 * (i & 7));
                }
#pragma unroll
                for (int q = 0; q < WORDS; ++q) args[(n * WORDS + q) * 64] = word[q];
                pairs += (unsigned)(w * w_p * __builtin_popcountll(here_too));
                lo_p = lo;
                w_p = w;
                v_pp = v_pn;
                alive = alive && least <= top_most;  // (a row with no cell of at most v: there is no such plan)
            }
            const bool ok = alive && W[0] <= top_most;
            tried[level] += __builtin_popcountll(__ballot(todo));
            const int ended = __builtin_popcountll(__ballot(ok));
            well[level] += ended;
            todo = todo && !ok;
            if (ended) {
                if (ok) a.C_out[a.stages ? c * S + xi - 1 : c] = W[0] >> K;
                int *bo = a.bounds_out + (a.stages ? c * tri + xi * (xi - 1) / 2 : c * S);
                const bool whole = (xi & 3) == 0 && ((uintptr_t)bo & 15) == 0;
                int at = 0, b[4] = {0, 0, 0, 0};
                for (int n = xi - 1; n >= 0; --n) {
                    const int e = (__builtin_amdgcn_readlane(v_row, n) & 0xffff) + at;
#pragma unroll
                    for (int u = 0; u < 4; ++u) b[u] = (n & 3) == u ? e : b[u];
                    if (ok && !whole) bo[n] = e;
                    if (ok && whole && (n & 3) == 0) *(int4 *)(bo + n) = make_int4(b[0], b[1], b[2], b[3]);
                    if (n) {
                        const unsigned word = args[(n * WORDS + (WORDS > 1 ? at >> 3 : 0)) * 64];
                        at = (int)(word >> (4 * (at & 7))) & 15;
                    }
                }
            }
        }
        open = open && !todo;
    }
#pragma unroll
    for (int level = 0; level < BAND_LEVELS; ++level) {
        if (pace.skip[level] > 0) --pace.skip[level];
        else if (8 * well[level] < tried[level]) pace.skip[level] = 7;
    }
    const unsigned long long left = __ballot((most >> lane & 1) && !open);
    // (a candidate that ended: its rows, of every stage count asked for)
    const unsigned long long rows = (unsigned long long)(__builtin_popcountll(__ballot(open)) * (a.stages ? tri - S : S - 1));
    if (lane == 0 && pairs) {
        auto &w = a.hdr->work[(c >> 6) & 63];
        atomicAdd(&w.pairs, pairs);
        atomicAdd(&w.band_pairs, pairs);
        atomicAdd(&w.rows, rows);
        atomicAdd(&w.band_rows, rows);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return left;
}

// How a row kernel for L <= 128 (A: dp_rows_args or dp_tile_args) passes by the candidates that bands finish: whole
// rows are computed for those left, a bit each in `left`.  Either a launch before this one has left them in memory,
// or (k_dp_rows) the ones with the channel-free plan are finished here, one per lane: where a wave's chunk is shorter
// than a wave is wide, the workgroup's candidates are dealt out together.  Else the chunk is taken in pieces of up to
// 64.  Where that has to be found out here and more than half of a piece is left, what follows it goes without.  (Bits
// that are in memory are read to the end: 270 000 orderings, L = 97, S = 11, 46 % of them left 1019 -> 801 us, 83 %
// 1216 -> 1164, all of them 1264 -> 1268.)
// (A kernel without this where neither can be worth it, pp_dp.hip.)  Returns whether all rows are to be computed.
template <int BANDS, typename A>
__device__ __forceinline__ bool band_begin(const A &a, unsigned char *smem, unsigned long long *&reach, unsigned long long &left) {
    reach = NULL;
    left = 0;
    if (BANDS == BAND_USE_NOT || a.g.band[band_top_at(a.S, 0, a.S)] < 0) return true;
    if (BANDS == BAND_USE_ALONE) return false;
    if constexpr (BANDS == BAND_USE_INSIDE) {
        if (!(a.pooled || a.links_at) || !band_free(a.g, a.g.band)) return true;
        unsigned long long *words = (unsigned long long *)(smem + (a.pooled ? 0 : a.links_at));
        reach = words + 4;
        band_links(a.g, a.g.band, reach);
        __syncthreads();
        if (a.pooled) {
            // dealt out together, before any wave needs its part of the LDS
            const int lane = threadIdx.x & 63, wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wpb = blockDim.x >> 6;
            const long long first = (long long)blockIdx.x * wpb * a.chunk;
            const int at = 64 * wib, total = (int)(a.N - first < wpb * a.chunk ? a.N - first : wpb * a.chunk);
            const unsigned long long word =
                at < total ? band_free_try(a.g, a.g.band, reach, first + at + lane, at + lane < total) : 0;
            if (lane == 0) words[wib] = word;
            __syncthreads();
            const int mine_at = wib * (int)a.chunk, w = mine_at >> 6, by = mine_at & 63;
            left = words[w] >> by;
            if (by && w + 1 < wpb) left |= words[w + 1] << (64 - by);
            left &= (1ull << a.chunk) - 1;
            __syncthreads();
        }
    }
    return false;
}

// The candidates base .. end - 1 of the chunk at c0: `left` of them, and where the piece ends.
template <int BANDS, typename A>
__device__ __forceinline__ int band_piece(const A &a, const unsigned long long *reach, long long c0, int base, int end,
                                          unsigned long long &left) {
    if constexpr (BANDS == BAND_USE_ALONE) {
        const unsigned long long *at = a.g.left + ((c0 + base) >> 6);
        const int by = (int)((c0 + base) & 63), n = end - base;
        left = at[0] >> by;
        if (by + n > 64) left |= at[1] << (64 - by);
        if (n < 64) left &= (1ull << n) - 1;
    } else if constexpr (BANDS == BAND_USE_INSIDE) {
        const int lane = threadIdx.x & 63;
        // (dealt out together: the chunk is one piece)
        if (!a.pooled) left = band_free_try(a.g, a.g.band, reach, c0 + base + lane, base + lane < end);
    }
    return end;
}

// L <= 128: the bands in launches of their own, in front of the DP kernel (links: room for D * D words).
int pp_launch_dp_band_alone(const dp_args &g, unsigned long long *links, unsigned long long *left, hipStream_t st);
