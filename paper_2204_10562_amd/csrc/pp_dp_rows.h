// Arguments and layout of the row kernel of the partition DP, 88 < L <= 128 (pp_dp_rows.hip).
#pragma once

#include "pp_common.h"
#include "pp_dp_generic.h"

#define DPR_PENDING 32  // candidates whose plans are written out together (one per lane)
// Backtrack rows a wave keeps before it must write plans out; one candidate needs up to S - 2.  (As many as
// leave four workgroups a compute unit at L = 128, S = 8; the stage-count search keeps more beside them:
// all 8! orderings, the whole search 142 us with 30 and three workgroups, 134 us with 23.)
__host__ __device__ static inline int dpr_arena_rows(int S, int stages) {
    return S > 32 ? 62 : stages && S <= 24 ? 23 : 30;
}
// Entries of a row (cells 0 .. L).  A wave writes 128 cells of a row, so what lies beyond L is in the row
// after it, which is written later.
__host__ __device__ static inline int dpr_stride(int L) { return L + 1; }
// Steps of a search in row n for a start.  With balanced stages a cell of row n chooses among the
// splits within P[l] / (n + 1) of it; a row that needs more gets a step more from then on.
__host__ __device__ static inline int dpr_steps(int L, int n) {
    int s = 1;
    while ((1 << s) - 1 < L / (n + 1) + L / (8 * (n + 1)) + 2) ++s;
    return s;
}
// Fewest rows a wave needs room for: 0 .. S-1, and while row n is computed its tables of minima in rows n ..
// n + steps - 1 (what those held is computed again after it).  With DPR_MAX_STEPS for the last row a search
// never takes a second round.
#define DPR_MAX_STEPS 7
static inline int dpr_min_rows(int L, int S) {
    int rows = S;
    for (int n = 1; n <= S - 2; ++n) {
        const int end = n + dpr_steps(L, n);
        rows = end > rows ? end : rows;
    }
    return rows;
}

struct dp_rows_args {
    int L, D, S, K;
    long long N;
    long long chunk;  // consecutive candidates walked by one wave
    int validate;     // orderings came from the caller: check them
    int rows;         // rows a wave has room for
    // LDS offset of a word per wave and the links' words (pp_dp_band.h; 0: no room for them); whether a workgroup's
    // candidates are dealt out together (chunks of less than 64: the words then take the waves' place)
    int links_at, pooled;
    int prio_left[3]; // priority k+1 while more than prio_left[k] candidates of the chunk are left
    dp_args g;        // tables, outputs and the generic fallback's arguments
};

// LDS bytes one wave needs: the key rows, the backtrack arena, the pending candidates' row slots and (for
// the stage-count search) the key of cell L of every row of the pending candidates; a row of 128 cells
// spills up to 128 - L entries.  (The workgroup adds the table of P.)
__host__ __device__ static inline size_t dpr_lds_per_wave(int L, int S, int rows, int stages) {
    const size_t spill = 128 - L, rs = dpr_stride(L);
    const size_t keys = (rows * rs + spill) * 4;
    const size_t arena = dpr_arena_rows(S, stages) * rs + spill;
    const size_t slots = (size_t)DPR_PENDING * S;
    const size_t tops = stages ? (size_t)DPR_PENDING * S * 4 : 0;
    return ((keys + tops + arena + slots) + 15) & ~(size_t)15;
}
#define DPR_TABLE ((64 + 129) * 4 + 128)  // bytes of the tables of P and of the runs of equal P

// Waves per workgroup, rows per wave and the workgroup's LDS for this shape (wpb == 0: it does not fit).
struct dpr_shape {
    int wpb, rows, waves_per_cu;
    size_t lds;
};
dpr_shape pp_dp_rows_shape(int L, int D, int S, int stages);

// grid workgroups of sh.wpb waves; wave w walks candidates [w*chunk, (w+1)*chunk)
int pp_launch_dp_rows(const dp_rows_args &a, int grid, const dpr_shape &sh, hipStream_t st);
