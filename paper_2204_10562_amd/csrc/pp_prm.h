// What the planner's kernels for replicated stages (pp_prm.hip, pp_prm_band.hip) share.
#pragma once

#include "pp_common.h"

struct prm_args {
    int L, D, M;
    int search;  // nonzero: the launch has LDS for the minima apart from the records
    long long N;
    const long long *fwd, *bwd, *actf, *actb, *alpha, *bw;
    const int *ord;  // [N][D]
    char *scratch;   // slots * slot_bytes
    size_t slot_bytes;
    int slots;
    long long *W_out;  // [N][D]: W of the best plan with xi stages at xi-1 (PP_INF64: none)
    int *bounds_out;   // [N][D(D+1)/2]
    int *reps_out;     // [N][D(D+1)/2]
    long long *pre_out;  // [3][L+1]: prefix sums of fwd, bwd, alpha for the kernels that follow
    int *band;           // header and tables of pp_prm_band.hip
    int32_t *status;
};

__host__ __device__ static inline int prm_states(int D) { return D * (D + 1) * (D + 2) / 6; }

// Index of state (i GPUs, xi stages, r replicas of the last stage), 1 <= xi <= i,
// 1 <= r <= i - xi + 1.
__host__ __device__ static inline int prm_sid(int i, int xi, int r) {
    return (i - 1) * i * (i + 1) / 6 + (xi - 1) * (i + 1) - xi * (xi - 1) / 2 + (r - 1);
}

__device__ __forceinline__ long long cdiv64(long long a, long long b) { return a / b + (a % b != 0); }

// Quotients of whole numbers below 2^53 by double arithmetic (instead of 64-bit integer division,
// about 100 instructions each).  `inv` is the reciprocal
// of den to 40 bits or more and the quotient is below 2^31, so the truncated product is off by one
// at most; the remainder (exact by the fused multiply-add) says which way.
__device__ __forceinline__ double prm_inv(double den) {
    const double r = __builtin_amdgcn_rcp(den);
    return __builtin_fma(r, __builtin_fma(-den, r, 1.0), r);
}
__device__ __forceinline__ int prm_ceil_div(double a, double den, double inv) {
    const double q = __builtin_trunc(a * inv), rem = __builtin_fma(-q, den, a);
    return (int)q + (rem > 0.0) + (rem > den);
}
__device__ __forceinline__ int prm_floor_div(double a, double den, double inv, int &rest) {
    const double q = __builtin_trunc(a * inv), rem = __builtin_fma(-q, den, a);
    const int up = rem >= den, down = rem < 0.0;
    rest = (int)(rem + (down ? den : up ? -den : 0.0));
    return (int)q + up - down;
}

// The bands (pp_prm_band.hip): ints of the header, then [D][L+1] pairs.
#define PRM_BAND_PARTS 0  // nonzero: every candidate is planned from bands of up to so many times a candidate's lanes,
#define PRM_BAND_LANES 1  // of which there are 8 or 16
#define PRM_BAND_MOST 1   // [i >= 1] (in LDS) float: most bytes over a cut of the states on i GPUs, there and back
#define PRM_BAND_LO 16    // [i >= 1] first cell of the states on i GPUs, and cells, in plans of three stages or more
#define PRM_BAND_W 32
#define PRM_BAND_LO2 48   // the same of the cuts of plans of two
#define PRM_BAND_W2 64
#define PRM_BAND_HDR 80
static inline size_t prm_band_bytes(int L, int D) { return (PRM_BAND_HDR + (size_t)D * (L + 1) * 2) * 4; }
// Most cells of a band with so many lanes per candidate: twice as many, or what lets three workgroups share the LDS
// of a compute unit (60 layers, 3000 orderings of 16 GPUs: 649 us for the call with two of them, 399 with three).
__host__ __device__ static inline int prm_band_cells(int D, int lanes) { return D > 12 ? 24 : 2 * lanes; }
// Ints of a row of Gmin, [stages before]: a multiple of 4, neighbouring rows in other banks.
__host__ __device__ static inline int prm_band_row(int D) { return ((D + 2) & ~3) | 4; }
// Bytes of a wave's states, per part (those on all GPUs are not kept); behind them the minima over the last stage's
// replicas, [GPUs, stages], and those over the links of ranks, [GPUs], which reading plans back takes.
__host__ __device__ static inline size_t prm_band_slot_bytes(int D) {
    return (size_t)prm_states(D - 1) * 64 * 6 + (size_t)(D * (D - 1) / 2 + D + 1) * 64 * 4;
}
static inline size_t prm_band_lds_bytes(int L, int D, int lanes, int waves) {
    const size_t wave = (size_t)(64 / lanes) * prm_band_cells(D, lanes) * (16 + prm_band_row(D) * 4) + 64 * 4;
    return (size_t)(L + 1) * (24 + 8 * D) + 16 + waves * wave + (size_t)D * D * 4 + PRM_BAND_HDR * 4;
}
// Waves of a workgroup: they share the tables that no candidate changes.
static inline int prm_band_waves(int L, int D, int lanes) {
    return prm_band_lds_bytes(L, D, lanes, 4) <= 64 * 1024 ? 4 : prm_band_lds_bytes(L, D, lanes, 2) <= 64 * 1024 ? 2 : 0;
}
// Whether a launch looks for bands.  A plan of M micro-batches is some 1 / M above the ideal (the AllReduce and the
// rounded quotients), and a band of 32 cells has room for 32 / L: with M = 4, 147 layers and 6 GPUs none is narrow
// enough, and to look costs 23 of 242 us.  (It does as well where links are slow, but not so slow that k_prm_prep sees it
// at once: 82 -> 104 us for 24 orderings of 4 GPUs, 60 layers, M = 16, with one link slower by 1000, 730 -> 767 for 24 of 12,
// 75, M = 24, with one slower by 30.  Where bands are narrow the same calls take 50 and 244 us.)
static inline bool prm_band_wanted(const prm_args &a) {
    return a.D >= 3 && a.L >= a.D && (long long)a.M * 32 >= a.L && (size_t)a.slots * a.slot_bytes >= 2 * prm_band_slot_bytes(a.D) &&
           prm_band_waves(a.L, a.D, 8) && prm_band_waves(a.L, a.D, 16);
}
// Enqueues the kernel that finds the bands and, behind it, the one that plans every candidate if they are narrow.
int pp_launch_prm_band(const prm_args &a, hipStream_t st);
