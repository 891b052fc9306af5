// One row of the partition DP by a wave, one lane per cell, a binary search per cell.
//
// Recursion for W(l, xi, r, i) of Sec. IV-B / the PRM listing with one replica per stage:
//   W[n][l] = min_{n<=k<l} max(g[k], P[l] - P[k]),   g[k] = max(W[n-1][k], X_n[k]),
// lowest minimising k kept.  Cells and splits are 32-bit keys (time << K) | k; times are compared
// in the keys' time field, P[k] as P[k] << K.
//
// With G(j) = min_{j<=k<l} g[k] the minimum is also min_j max(G(j), P[l] - P[j]).  G rises with j
// and P[l] - P[j] falls, so it lies at their crossing: the first split j >= n that is not done for,
// where j is done for iff P[l] - P[j] > G(j+1).  W[n][l] = max(G(j), P[l] - P[j]); where P rises
// strictly every split left of j is worse (its difference term is above G(j) and above j's), and
// the lowest best split is j if g[j] does not exceed that value, else the first one after j that
// does not.
//
// G depends on the cell through its upper end l.  The search ignores that: it uses the minima over
// all splits up to the end of the row, H(j) = min_{k>=j} g[k], so that one pass over the row
// (row_build, right to left) leaves h[j] = H(j+1) + P[j] for all cells, and the search is for the
// first j >= n with h[j] >= P[l] (or j = l-1): one LDS read per step.  What it finds is exact
// whenever g[j] <= H(j+1), i.e. nothing later undercuts split j: then G(j) = g[j] = H(j), and W =
// max(g[j], P[l] - P[j]).  That is almost always so where links are fast (W[n-1] rises, and few
// transfers put peaks into g).  Otherwise (the crossing is on a peak) a split after j and before l that
// attains H(j+1) proves G(j) = H(j) too, and it is the answer; failing that the undercutting split
// is not the cell's yet, and the cell looks at its splits one by one from l-1 leftwards until the
// difference term alone exceeds the best value: 0..4 % of the cells with links from 10 GB/s, for 4..10
// splits each.  Rows with many such splits (row_build counts them) are searched by row_jump instead.
//
// Zero-length layers (strict == 0): P is equal at neighbouring cuts, and a split left of j with the
// same P can tie; the lowest split of the run of equal P whose g does not exceed the value is kept.
#pragma once

#include "pp_common.h"

#define DPP_ROW_SHL(n) (0x100 + (n))

__device__ __forceinline__ int row_imin(int a, int b) { return a < b ? a : b; }
__device__ __forceinline__ int row_imax(int a, int b) { return a > b ? a : b; }

__device__ __forceinline__ void row_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// LDS through 32-bit addresses, so that a search can carry the address it reads.
typedef __attribute__((address_space(3))) unsigned row_lds;
__device__ __forceinline__ int row_addr(const void *p) { return (int)(unsigned)(uintptr_t)(const row_lds *)p; }
__device__ __forceinline__ unsigned row_at(int addr) { return *(const row_lds *)(uintptr_t)(unsigned)addr; }

struct dp_row {
    const int *W;   // W[n-1][k], k = 0 ..
    int *g;         // g[k] (may be W itself)
    unsigned *h;    // h[j], j = -1 .. (an entry of padding in front)
    int *out;       // W[n][l]
    const int *PK;  // (P[k] << K) - k, k = -1 .. (an entry of padding in front; P[L] beyond L)
    int n, L, K, kmask, steps;
    bool strict;
    int lane;
    int carry;   // min g over the splits to the right of what row_build has done
    int falls;   // splits whose g a later one undercuts, as far as row_build has looked
    int again;   // rounds of `steps` steps the searches took beyond the first, over all chunks of 64 cells
};

// Whether P rises strictly (PK as above); once per wave: the preparation kernel, which could leave it in
// the workspace header, is on the path of calls that never search (7.6 against 7.4 us).
__device__ __forceinline__ bool row_is_strict(const int *PK, int L, int lane) {
    bool rises = true;
    for (int k = lane; k < L; k += 64) rises &= PK[k + 1] + 1 > PK[k];
    return __ballot(!rises) == 0;
}

// Once per wave, with everything above but W, g, out and n set: whether P rises strictly, and what row_build
// does not write where the last chunk ends with the row (L a multiple of 64): nothing is right of split
// L - 1, so nothing undercuts it.
__device__ __forceinline__ void row_begin(dp_row &r) {
    r.strict = row_is_strict(r.PK, r.L, r.lane);
    if (r.lane == 0) r.h[r.L - 1] = (unsigned)(PP_INF32 & ~r.kmask) + (unsigned)(r.PK[r.L - 1] + (r.L - 1));
    row_lds_sync();
}

// Steps of a search in row n for a start.  With balanced stages a cell of row n chooses among the
// splits within P[l] / (n + 1) of it; a row that needs more gets a step more from then on.
__device__ __forceinline__ int row_first_steps(int L, int n) {
    int s = 1;
    while ((1 << s) - 1 < L / (n + 1) + L / (8 * (n + 1)) + 2) ++s;
    return s;
}

// Minima over the lanes from each lane on (and over `carry`).
__device__ __forceinline__ int row_suffix_min(int v, int carry, int lane) {
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_SHL(1), 0xf, 0xf, false));
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_SHL(2), 0xf, 0xf, false));
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_SHL(4), 0xf, 0xf, false));
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_SHL(8), 0xf, 0xf, false));
    const int s3 = row_imin(__builtin_amdgcn_readlane(v, 48), carry);
    const int s2 = row_imin(__builtin_amdgcn_readlane(v, 32), s3);
    const int s1 = row_imin(__builtin_amdgcn_readlane(v, 16), s2);
    int right = carry;
    right = lane < 48 ? s3 : right;
    right = lane < 32 ? s2 : right;
    right = lane < 16 ? s1 : right;
    return row_imin(v, right);
}

// Splits c0 .. c0 + 64 U - 1, after everything to their right: g and h.  xv: the link's times; w
// receives W[n-1] of these splits.  (All loads before all stores: the compiler cannot tell the
// arrays apart and would wait for each load in turn.)
template <int U>
__device__ __forceinline__ void row_build(dp_row &r, int c0, const int *xv, int (&w)[U]) {
    int g[U], pk[U];
    const int k0 = c0 + r.lane;
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = r.W[k0 + 64 * u];
#pragma unroll
    for (int u = 0; u < U; ++u) pk[u] = r.PK[k0 + 64 * u - 1];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = k0 + 64 * u;
        const int xk = (int)((unsigned)xv[u] << r.K) | k, wk = (w[u] & ~r.kmask) | k;
        g[u] = row_imax(wk, xk);
        if (u == 0) g[u] = k < r.n ? k : g[u];          // (splits below n: small, so that g rises over them)
        if (u == U - 1) g[u] = k < r.L ? g[u] : PP_INF32;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) r.g[k0 + 64 * u] = g[u];
#pragma unroll
    for (int u = U - 1; u >= 0; --u) {
        int m = g[u];
        const int next = __builtin_amdgcn_update_dpp(r.carry, g[u], DPP_WAVE_SHL1, 0xf, 0xf, false);
        const unsigned long long falls = __ballot(next < m);
        r.falls += __builtin_popcountll(falls);
        if (falls) m = row_suffix_min(m, r.carry, r.lane);
        r.carry = __builtin_amdgcn_readlane(m, 0);
        g[u] = m;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = k0 + 64 * u;
        r.h[k - 1] = (unsigned)(g[u] & ~r.kmask) + (unsigned)(pk[u] + (k - 1));
    }
}

// The cell whose crossing lies on a peak or, where layers have length zero, on a split that shares its P
// with the one before.
__device__ __forceinline__ int row_on_peak(const dp_row &r, int j, int l, unsigned Pl) {
    const unsigned t = ~(unsigned)r.kmask, Pj = (unsigned)(r.PK[j] + j);
    const unsigned d = Pl - Pj, gj = (unsigned)r.g[j] & t, nx = r.h[j] - Pj;
    const bool alive = gj <= nx;
    const unsigned m = alive ? gj : nx, v = d > m ? d : m;
    int a = j;
    if (!r.strict)
        while (a > r.n && (unsigned)(r.PK[a - 1] + a - 1) == Pj) --a;
    // If split j or a later one of the cell attains H(j), the first with g <= v is the answer.  (Four
    // splits per trip to LDS; the row has entries beyond L.)
    int e = alive ? j : j + 1;
    if (!alive)
        for (bool look = true; look && e < l;) {
            unsigned x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = (unsigned)r.g[row_imin(e + i, r.L)] & t;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                look = look && x[i] > nx;
                e += look;
            }
        }
    if (e < l) {
        while (a < e && ((unsigned)r.g[a] & t) > v) ++a;
        return (int)v | a;
    }
    int best = PP_INF32;
    for (int k = l - 1; k >= r.n; k -= 4) {
        int x[4], dk[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = row_imax(k - i, r.n);
            x[i] = r.g[at];
            dk[i] = (int)(Pl - (unsigned)r.PK[at]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) best = row_imin(best, row_imax(x[i], dk[i]));
        if ((dk[3] & ~r.kmask) > (best & ~r.kmask)) break;
    }
    return best;
}

// One step of U searches: back by s bytes where that split is not done for (CLAMP: not below `low`).
template <int U, bool CLAMP>
__device__ __forceinline__ void row_step(int s, int (&pos)[U], const unsigned (&Pl)[U], int low) {
    int j[U];
    unsigned hv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        j[u] = CLAMP ? row_imax(pos[u] - s, low) : pos[u] - s;
        hv[u] = row_at(j[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) pos[u] = hv[u] >= Pl[u] ? j[u] : pos[u];
}

// Cells c0 + 1 .. c0 + 64 U (cells beyond L repeat cell L, those up to n are infinite).
// w receives them too.
template <int U>
__device__ __forceinline__ void row_search(dp_row &r, int c0, int (&w)[U]) {
    int pos[U];
    unsigned Pl[U];
    const int h0 = row_addr(r.h), low = h0 + 4 * r.n, reach = (4 << r.steps) - 4;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = c0 + 64 * u + r.lane;
        Pl[u] = (unsigned)(r.PK[k + 1] + (k + 1));
        pos[u] = h0 + 4 * row_imin(k, r.L - 1);
    }
    const int limit = 4 * (c0 - r.n);
    for (bool first = true;; first = false) {
        int from[U];
#pragma unroll
        for (int u = 0; u < U; ++u) from[u] = pos[u];
        // (loops: straight-line code entered at the first step was measured 5 % slower)
        if (first && limit >= reach) {
            for (int s = 2 << r.steps; s >= 4; s >>= 1) row_step<U, false>(s, pos, Pl, low);  // no lane can get below split n
        } else {
            for (int s = 2 << r.steps; s >= 4; s >>= 1) row_step<U, true>(s, pos, Pl, low);
        }
        bool more = false;
#pragma unroll
        for (int u = 0; u < U; ++u) more |= pos[u] > low && pos[u] == from[u] - reach;
        if (!__ballot(more)) break;
        r.again += U;
    }
    const int to_g = row_addr(r.g) - h0, to_pk = row_addr(r.PK) - h0;
    unsigned gv[U], pv[U], hv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { gv[u] = row_at(pos[u] + to_g); pv[u] = row_at(pos[u] + to_pk); hv[u] = row_at(pos[u]); }
    bool odd = false, peak[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        w[u] = row_imax((int)gv[u], (int)(Pl[u] - pv[u]));
        peak[u] = gv[u] + pv[u] > hv[u];  // g[j] > H(j+1), the key's low bits being j on both sides
    }
    if (!r.strict) {
        // splits left of j tie only where they have its P
#pragma unroll
        for (int u = 0; u < U; ++u) peak[u] |= row_at(pos[u] + to_pk - 4) == pv[u] + 1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) odd |= peak[u] && (u || c0 + r.lane >= r.n);
    if (__ballot(odd)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = c0 + 64 * u + r.lane + 1;
            if (peak[u] && l > r.n && l <= r.L) w[u] = row_on_peak(r, (pos[u] - h0) >> 2, l, Pl[u]);
        }
    }
    w[0] = c0 + r.lane >= r.n ? w[0] : PP_INF32;
#pragma unroll
    for (int u = 0; u < U; ++u) r.out[c0 + 64 * u + r.lane + 1] = w[u];
}

// Rows in which g falls often (links that bind): what undercuts a split lies beyond the cell then, and the
// search above would send most cells to row_on_peak.  The same crossing with minima that end at the cell:
// back from split l - 1 by 16, 4 and 1 while the split in front costs no more than the least g in between
// (pp_dp_rows.hip has the reasoning; keys for times).  T16[j] = min g[j+1 .. j+16] in the place of h and
// T4[j] = min g[j+1 .. j+4] in the row being produced, both 0 for j < n; the row's cells are therefore
// worked out from the right, where they overwrite what no cell left of them needs.
__device__ __forceinline__ void row_tables(const dp_row &r) {
    row_lds_sync();
    for (int j = r.lane; j < r.L; j += 64) {
        const int a = r.g[j + 1], b = r.g[j + 2], c = r.g[j + 3], d = r.g[j + 4];
        r.out[j] = j < r.n ? 0 : row_imin(row_imin(a, b), row_imin(c, d));
    }
    row_lds_sync();
    for (int j = r.lane; j < r.L; j += 64) {
        const int a = r.out[j], b = r.out[j + 4], c = r.out[j + 8], d = r.out[j + 12];
        r.h[j] = (unsigned)row_imin(row_imin(a, b), row_imin(c, d));
    }
    row_lds_sync();
}

// Cells c0 + 1 .. c0 + 64 U; returns the trips to LDS it took.
template <int U>
__device__ __forceinline__ int row_jump(const dp_row &r, int c0) {
    int pos[U];
    unsigned low[U], Pl[U];
    const int p0 = row_addr(r.PK), to_16 = row_addr(r.h) - p0, to_4 = row_addr(r.out) - p0, to_g = row_addr(r.g) - p0;
    const int first = p0 + 4 * r.n;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int k = c0 + 64 * u + r.lane;
        Pl[u] = (unsigned)(r.PK[k + 1] + (k + 1));
        pos[u] = p0 + 4 * row_imin(k, r.L - 1);
        low[u] = PP_INF32;
    }
    // (split 0 stands for all in front of it: its minima are 0)
    auto step = [&](int by, int to, bool check) {
        int j[U];
        unsigned p[U], q[U];
        bool any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) { j[u] = row_imax(pos[u] - by, p0); p[u] = row_at(j[u]); q[u] = row_at(j[u] + to); }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned m = q[u] < low[u] ? q[u] : low[u];
            const bool back = Pl[u] - p[u] < m && (!check || j[u] >= first);
            pos[u] = back ? j[u] : pos[u];
            low[u] = back ? m : low[u];
            any |= back;
        }
        return any;
    };
    int trips = 7;
    while (__ballot(step(64, to_16, false))) ++trips;
    for (int i = 0; i < 3; ++i) step(16, to_4, false);
    for (int i = 0; i < 3; ++i) step(4, to_g + 4, true);
    int w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = row_imin((int)low[u], row_imax((int)row_at(pos[u] + to_g), (int)(Pl[u] - row_at(pos[u]))));
    if (!r.strict) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = (pos[u] - p0) >> 2;
            int a = j;
            while (a > r.n && r.PK[a - 1] + (a - 1) == r.PK[j] + j) --a;
            while (a < j && (r.g[a] | r.kmask) > (w[u] | r.kmask)) ++a;
            w[u] = a < j ? (w[u] & ~r.kmask) | a : w[u];
        }
    }
    row_lds_sync();
    w[0] = c0 + r.lane >= r.n ? w[0] : PP_INF32;
#pragma unroll
    for (int u = 0; u < U; ++u) r.out[c0 + 64 * u + r.lane + 1] = w[u];
    return trips;
}
