// The bands of pp_dp_band.h for L > 128, around the preparation of pp_share.hip: every candidate that ends well
// here is finished, the others go to k_dp_big.
//
// First pass (before the keys; where the link classes do not fit the table of keys): all candidates.  Those left
// are counted into the buckets of their first devices, in whose order k_dp_big takes them.  Second pass (the
// list of representatives is there): the representatives; where there are none, what the first pass left takes
// its places in the order of the buckets.
//
// What bounds it: trips to memory with few waves, seven a compute unit by LDS.  Where the channel-free plan is the answer
// these are the orderings read and the plans written (2^20 candidates of 32 stages: 268 MB in 215 us, vector units busy 22 % of
// the time, 1.6 waves per SIMD in flight); else a row's gather (one vector load per lane from its link's row) and, with bands of
// many cells, the pairs, 1.5 vector instructions each for 64 candidates at once (200 000 candidates, L = 300, S = 16, that end in
// the second level: 276 us, busy 40 %).
#include "pp_dp_band.h"
#include "pp_share.h"

struct band_args {
    dp_args g;
    const int *band;                  // NULL: every candidate is left
    unsigned long long *links;        // band_links' words, or NULL
    int *keys, *table, *reps;
    unsigned long long *left;         // BAND_ALONE: a bit per candidate
};

enum { BAND_FIRST, BAND_SECOND, BAND_ALONE };
template <int PASS>
__global__ __launch_bounds__(64) void k_dp_band(band_args b) {
    constexpr bool FIRST = PASS == BAND_FIRST;
    extern __shared__ __align__(16) unsigned char smem[];
    const dp_args &a = b.g;
    const int S = a.S, D = a.D, L = a.L, lane = threadIdx.x;
    const bool active = PASS != BAND_ALONE && share_table_size(a.hdr->share_nc, S) != 0;
    int kdev = 0;
    if (PASS != BAND_ALONE && !active) share_buckets(D, S, kdev);
    if (FIRST ? active || !kdev : PASS == BAND_SECOND && !active && !a.hdr->share_npend) return;
    if (PASS == BAND_SECOND && !active) {
        // counting sort, last step: every candidate left takes the next free position of its bucket
        for (long long c = (long long)blockIdx.x * 64 + lane; c < a.N; c += (long long)gridDim.x * 64) {
            const int key = b.keys[c];
            if (key >= 0) b.reps[atomicAdd(&b.table[key], 1)] = (int)c;
        }
        return;
    }
    if (pp_is_flat(a.hdr) || !(pp_vmax(a.hdr) < a.fit_limit)) return;  // (the DP kernel looks at all candidates)
    const bool use = b.band != NULL && b.band[band_top_at(S, 0, S)] >= 0;
    const unsigned long long *links = use && band_free(a, b.band) ? b.links : NULL;
    if (!FIRST && !use) return;
    int *PK = (int *)(smem + band_lds_per_wave(S));
    if (use)
        for (int k = lane; k < L + 1 + BAND_CELLS; k += 64) PK[k] = (a.p32[k < L ? k : L] << a.K) - k;
    __syncthreads();
    band_pace pace = {};
    const long long todo = PASS != BAND_SECOND ? a.N : (long long)a.hdr->share_nsorted;
    const bool cells = todo >= a.band_all;
    if (PASS == BAND_SECOND && !cells && !links) return;
    for (long long r = (long long)blockIdx.x * 64; r < todo; r += (long long)gridDim.x * 64) {
        const bool live = r + lane < todo;
        const long long c = live ? (PASS != BAND_SECOND ? r + lane : b.reps[r + lane]) : 0;
        unsigned long long left = __ballot(live);
        if (use) left = cells ? band_try(a, b.band, links, PK, smem, c, live, pace) : band_free_try(a, b.band, links, c, live);
        if (PASS == BAND_ALONE) {
            if (lane == 0) b.left[r >> 6] = left;
            continue;
        }
        const bool mine = left >> lane & 1;
        if (FIRST) {
            if (live) {
                unsigned key = 0;
                if (mine) {
                    const int *row = a.ord + c * S;
                    for (int n = 0; n < kdev; ++n) {
                        int d = row[n];
                        d = (d < 0 || d >= D) ? 0 : d;  // (a bad row is found by the DP kernel; any bucket will do)
                        key = key * (unsigned)D + (unsigned)d;
                    }
                    // (the table starts at SHARE_NONE everywhere: counts are relative to that, unsigned)
                    atomicAdd((unsigned *)&b.table[key], 1u);
                }
                b.keys[c] = mine ? (int)key : -1;
            }
            if (left && lane == 0) atomicAdd(&a.hdr->share_npend, (unsigned)__builtin_popcountll(left));
        } else if (live && !mine) {
            b.keys[c] |= SHARE_ENDED;
        }
    }
}

// Every link's words, one wave per link.
__global__ __launch_bounds__(256) void k_band_links(band_args b) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i < b.g.D * b.g.D) band_link_wave(b.g, b.band, i, b.links);
}

static band_args band_base(const dp_args &g, const int *band, unsigned long long *links) {
    band_args b = {};
    b.g = g;
    b.band = band;
    b.links = links;
    return b;
}

template <int PASS>
static int launch_band(const band_args &b, hipStream_t st) {
    // (workgroups of one wave, a few groups of candidates each where there are many: see band_pace)
    const long long groups = (b.g.N + 63) / 64;
    const dim3 grid((unsigned)(groups < 2048 ? groups : 2048));
    const size_t lds = band_lds_per_wave(b.g.S) + (size_t)(b.g.L + 1 + BAND_CELLS) * 4;
    hipLaunchKernelGGL(k_dp_band<PASS>, grid, dim3(64), lds, st, b);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}

int pp_launch_dp_band(const dp_args &g, const int *band, unsigned long long *links, int *keys, int *table, int *reps,
                      int first, hipStream_t st) {
    band_args b = band_base(g, band, links);
    b.keys = keys;
    b.table = table;
    b.reps = reps;
    return first ? launch_band<BAND_FIRST>(b, st) : launch_band<BAND_SECOND>(b, st);
}

int pp_launch_dp_band_alone(const dp_args &g, unsigned long long *links, unsigned long long *left, hipStream_t st) {
    band_args b = band_base(g, g.band, links);
    b.left = left;
    if (b.links) hipLaunchKernelGGL(k_band_links, dim3((g.D * g.D + 3) / 4), dim3(256), 0, st, b);
    return launch_band<BAND_ALONE>(b, st);
}
