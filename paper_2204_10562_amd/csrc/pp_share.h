// What the preparation of shared DPs (pp_share.hip) and the pass over the bands (pp_dp_band.hip) both need.
#pragma once

#include "pp_common.h"
#include "pp_dp_generic.h"

#define SHARE_NONE 0x7fffffff
// Set in a representative's key (below 2^20) once its plan is there.
#define SHARE_ENDED 0x40000000

// Keys of S - 1 digits in base nc: how many there are, 0 if they do not fit the table.
__host__ __device__ __forceinline__ unsigned share_table_size(unsigned nc, int S) {
    if (nc == 0) return S > 1 ? 0 : 1;
    unsigned tsize = 1;
    for (int n = 1; n < S && tsize; ++n) {
        const unsigned long long t = (unsigned long long)tsize * nc;
        tsize = t <= PP_SHARE_TABLE ? (unsigned)t : 0;
    }
    return tsize;
}

// Buckets of the first kdev devices that fit the table (kdev = 0: fewer than two, or there is no row to share).
__device__ __forceinline__ unsigned share_buckets(int D, int S, int &kdev) {
    unsigned nbuck = 1;
    kdev = 0;
    while (kdev < S && (unsigned long long)nbuck * (unsigned)D <= PP_SHARE_TABLE) { nbuck *= (unsigned)D; ++kdev; }
    if (kdev < 2 || S < 3) kdev = 0;
    return nbuck;
}

// The two passes of pp_dp_band.hip (band: the pack kernel's table, or NULL; links: of k_share_classes).
int pp_launch_dp_band(const dp_args &g, const int *band, unsigned long long *links, int *keys, int *table, int *reps,
                      int first, hipStream_t st);
