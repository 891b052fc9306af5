// The bands of pp_dp_band.h for L > 128, around the preparation of pp_share.hip: every candidate that ends well
// here is finished, the others go to k_dp_big.
//
// First pass (before the keys; where the link classes do not fit the table of keys): all candidates.  Those left
// are counted into the buckets of their first devices, in whose order k_dp_big takes them.  Second pass (the
// list of representatives is there): the representatives; where there are none, what the first pass left takes
// its places in the order of the buckets.
//
// What bounds it: trips to memory with few waves, seven a compute unit by LDS.  Where the channel-free plan is the answer and
// the plans are asked for these are the orderings read and the plans written (2^20 candidates of 32 stages: 268 MB in 215 us,
// vector units busy 22 % of the time, 1.6 waves per SIMD in flight); else a row's gather (one vector load per lane from its link's row) and, with bands of
// many cells, the pairs, 1.5 vector instructions each for 64 candidates at once (200 000 candidates, L = 300, S = 16, that end in
// the second level: 276 us, busy 40 %).
#include "pp_dp_band.h"
#include "pp_makespan_path.h"
#include "pp_share.h"

struct band_args {
    dp_args g;
    const int *band;                  // NULL: every candidate is left
    unsigned long long *links;        // band_links' words, or NULL
    int *keys, *table, *reps;
    unsigned long long *left;         // BAND_ALONE: a bit per candidate
    int first;                        // L > 128: candidates are taken only where no representatives are
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
    const bool looked = PASS != BAND_SECOND && a.fx && a.hdr->free_valid;
    for (long long r = (long long)blockIdx.x * 64; r < todo; r += (long long)gridDim.x * 64) {
        const bool here = r + lane < todo, live = here && !(looked && (a.fbits[r >> 6] >> lane & 1));
        const long long c = here ? (PASS != BAND_SECOND ? r + lane : b.reps[r + lane]) : 0;
        unsigned long long left = __ballot(live);
        if (PASS != BAND_ALONE && looked && !left) continue;
        if (use && left) left = cells ? band_try(a, b.band, links, PK, smem, c, live, pace) : band_free_try(a, b.band, links, c, live);
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

// The candidates with the channel-free plan, scheduled where they are found (a.fx; one per lane).  Every stage is then
// the same for all, and a link's times come from the few at the plan's cuts: one load per stage, of a table by stage and
// link, which also says whether the link reaches into its row.  Candidates that have another plan are left to
// k_dp_band (a bit per candidate that is not).
// What bounds it: instruction issue (71 vector instructions per stage), then the orderings' bytes.  2^20 candidates of 32
// stages, one count: 127 us, where the look for the plan (which also wrote 134 MB of bounds) took 215 and the schedules, whose
// transfer times lie a cache line apart in [link][cut], 388; the whole call 720 -> 260 us.  20 011 of 48 stages 167 -> 142,
// 200 003 of 11, two counts 75 -> 59.
template <int NM>
__global__ __launch_bounds__(256) void k_band_free(band_args b) {
    const dp_args &a = b.g;
    const int S = a.S, D = a.D, tid = threadIdx.x, lane = tid & 63, nl = D * D;
    if (b.first) {
        int kdev = 0;
        if (share_table_size(a.hdr->share_nc, S) != 0) return;
        share_buckets(D, S, kdev);
        if (!kdev) return;
    }
    if (pp_is_flat(a.hdr) || !(pp_vmax(a.hdr) < a.fit_limit)) return;
    if (b.band[band_top_at(S, 0, S)] < 0 || !band_free(a, b.band)) return;
    int M[NM], mmax = 1;
    bool briefly[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) {
        M[q] = a.f_Ms[q];
        mmax = M[q] > mmax ? M[q] : mmax;
    }
    mk_briefly<PP_SCHED_PE>(M, S, briefly);
    const int C = b.band[band_C_at(S, S)];
    if (C > pp_time_limit(mmax, S)) return;
    if (blockIdx.x == 0 && tid == 0) a.hdr->free_valid = 1;
    // lane n: the passes of stage n
    const int *plan = b.band + band_plan_at(S, S);
    const int e0 = lane > 0 && lane < S ? plan[lane - 1] : 0, e1 = lane < S ? plan[lane] : a.L;
    const int v_F = (int)(a.PF[e1] - a.PF[e0]), v_B = (int)(a.PB[e1] - a.PB[e0]);
    const long long groups = (a.N + 63) / 64;
    const int waves = blockDim.x >> 6;
    for (long long g = (long long)blockIdx.x * waves + __builtin_amdgcn_readfirstlane(tid >> 6); g < groups; g += (long long)gridDim.x * waves) {
        const long long c = g * 64 + lane;
        const bool live = c < a.N;
        const int *row = a.ord + (live ? c : a.N - 1) * S;
        bool bad = false, reach = false;
        unsigned long long seen = 0;
        int before = 0, differs = lane ? S : 0;  // the first place where the devices differ from those of the lane before
        mk_path<int, NM> path;
        path.start();
        struct four { int2 x[4]; int d[4]; };
        // (rows of four devices at a time; the last of a row that is no multiple of four overlap with those before)
        auto devices = [&](int n0) {
            band_int4 v;
            if (S >= 4) {
                const int at = n0 + 4 <= S ? n0 : S - 4;
                v = *(const band_int4 *)(row + at);
                for (int s = n0 - at; s > 0 && s < 4; --s) { v.v[0] = v.v[1]; v.v[1] = v.v[2]; v.v[2] = v.v[3]; }
            } else {
                for (int u = 0; u < 4; ++u) v.v[u] = u < S ? row[u] : 0;
            }
            return v;
        };
        auto links = [&](four &f, const band_int4 &v, int n0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int n = n0 + u;
                int d = v.v[u];
                f.x[u] = make_int2(0, 0);
                f.d[u] = d;
                if (n >= S) continue;
                if (a.validate) {
                    bad |= d < 0 || d >= D;
                    d = bad ? 0 : d;
                    bad |= (seen >> d) & 1;
                    seen |= 1ull << d;
                }
                if (n) f.x[u] = a.fx[n * nl + before * D + d];
                before = d;
            }
        };
        four now, then;
        band_int4 v = devices(0);
        links(now, v, 0);
        if (S > 4) v = devices(4);
        for (int n0 = 0; n0 < S; n0 += 4) {
            if (n0 + 4 < S) {
                links(then, v, n0 + 4);
                if (n0 + 8 < S) v = devices(n0 + 8);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int n = n0 + u;
                if (n >= S) continue;
                const int o = __builtin_amdgcn_update_dpp(now.d[u], now.d[u], DPP_WAVE_SHR1, 0xf, 0xf, false);
                differs = now.d[u] != o && differs == S ? n : differs;
                reach |= now.x[u].x < 0;
                mk_stage<PP_SCHED_PE>(path, n, S, __builtin_amdgcn_readlane(v_F, n), __builtin_amdgcn_readlane(v_B, n),
                                      now.x[u].x & 0x7fffffff, now.x[u].y, M, briefly);
            }
            now = then;
        }
        const bool done = live && !bad && !reach;
        const unsigned long long ended = __ballot(done);
        if (done) {
            if (b.first) b.keys[c] = -1;
            a.C_out[c] = C;
#pragma unroll
            for (int q = 0; q < NM; ++q)
                if (q < a.f_nM && a.fT) a.fT[(long long)q * a.N + c] = path.longest(q);
        }
        // (rows of neighbours in the wave that begin with the same devices count once, the last row for everyone)
        const bool after = lane && (ended >> (lane - 1) & 1);
        int rows = done ? 1 + band_max(0, S - 1 - (after && differs > 1 ? differs : 1)) : 0;
        // (and the least time of the group, lowest candidate first; a loop, because what a wave runs once waits for its
        // instructions: unrolled, 20 011 candidates of 48 stages take 26.2 instead of 25.3 us)
        int T[NM], least[NM];
#pragma unroll
        for (int q = 0; q < NM; ++q) least[q] = T[q] = done ? path.longest(q) : 0x7fffffff;
#pragma unroll 1
        for (int off = 32; off; off >>= 1) {
            rows += __shfl_xor(rows, off);
#pragma unroll
            for (int q = 0; q < NM; ++q) least[q] = band_min(least[q], __shfl_xor(least[q], off));
        }
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const unsigned long long at = __ballot(T[q] == least[q]) & ended;
            if (q < a.f_nM && lane == 0) a.fleast[q * groups + g] = at ? (long long)least[q] << 6 | __builtin_ctzll(at) : -1;
        }
        if (lane == 0) {
            a.fbits[g] = ended;
            if (rows) {
                auto &w = a.hdr->work[g & 63];
                atomicAdd(&w.rows, (unsigned long long)rows);
                atomicAdd(&w.free_rows, (unsigned long long)rows);
            }
        }
    }
}

static int launch_free(const band_args &b, hipStream_t st) {
    if (!b.g.fx || !b.band || !b.links) return PP_OK;
    const long long blocks = (b.g.N + 255) / 256;
    const dim3 grid((unsigned)(blocks < 2048 ? blocks : 2048));
    if (b.g.f_nM == 1) hipLaunchKernelGGL(k_band_free<1>, grid, dim3(256), 0, st, b);
    else if (b.g.f_nM == 2) hipLaunchKernelGGL(k_band_free<2>, grid, dim3(256), 0, st, b);
    else hipLaunchKernelGGL(k_band_free<PP_FREE_COUNTS>, grid, dim3(256), 0, st, b);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
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
    if (!first) return launch_band<BAND_SECOND>(b, st);
    b.first = 1;
    const int rc = launch_free(b, st);
    return rc ? rc : launch_band<BAND_FIRST>(b, st);
}

int pp_launch_dp_band_alone(const dp_args &g, unsigned long long *links, unsigned long long *left, hipStream_t st) {
    band_args b = band_base(g, g.band, links);
    b.left = left;
    if (b.links) hipLaunchKernelGGL(k_band_links, dim3((g.D * g.D + 3) / 4), dim3(256), 0, st, b);
    const int rc = launch_free(b, st);
    return rc ? rc : launch_band<BAND_ALONE>(b, st);
}
