// Arguments of the partition DP kernel for 88 < L <= 128 (pp_dp_rows.hip).
#pragma once

#include "pp_common.h"
#include "pp_dp_generic.h"

#define DPR_PENDING 32  // candidates whose plans are written out together (one per lane)
// Backtrack rows a wave keeps before it must write plans out; one candidate needs up to S - 2.
__host__ __device__ static inline int dpr_arena_rows(int S) { return S <= 32 ? 32 : 64; }
#define DPR_RS (128 + 4)  // entries of a row

struct dp_rows_args {
    int L, D, S, K;
    long long N;
    long long chunk;  // consecutive candidates walked by one wave
    int validate;     // orderings came from the caller: check them
    int prio_left[3]; // priority k+1 while more than prio_left[k] candidates of the chunk are left
    dp_args g;        // tables, outputs and the generic fallback's arguments
};

// LDS bytes one wave needs: S key rows, g and h of one row, the key of cell L of every row of the
// pending candidates (used by the stage-count search only), the backtrack arena, and the pending
// candidates' row slots.  (The workgroup adds one row: the table of P.)
__host__ __device__ static inline size_t pp_dp_rows_lds_per_wave(int S) {
    size_t rows = (size_t)(S + 2) * DPR_RS * 4;
    size_t tops = (size_t)DPR_PENDING * S * 4;
    size_t arena = (size_t)dpr_arena_rows(S) * DPR_RS;
    size_t slots = (size_t)DPR_PENDING * S;
    return (rows + tops + arena + slots + 15) & ~(size_t)15;
}

// grid workgroups of wpb waves; wave w walks candidates [w*chunk, (w+1)*chunk)
int pp_launch_dp_rows(const dp_rows_args &a, int grid, int wpb, hipStream_t st);
