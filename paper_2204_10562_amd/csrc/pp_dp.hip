// pp_partition_dp: min-max partition of L layers into S contiguous stages, one candidate
// device ordering per workgroup.
//
// Recursion for W(l, xi, r, i) of Sec. IV-B / the PRM listing with one replica per stage:
//   W[0][l] = P[l];  W[n][l] = min_{n<=k<l} max(W[n-1][k], X_n[k], P[l] - P[k]),
// lowest minimising k kept, plan read back from (S-1, L).
//
// Two representations.  When every time is below 2^(31-K) - 1 (K = bits of a split index) a
// cell is a 32-bit key (time << K) | k: the max of two keys whose low bits both equal k keeps
// k, so a plain integer min over k yields the smallest time and, among equal times, the
// lowest k - the required tie-break - at three integer operations per (cell, split) pair.
// Otherwise cells are int64 with an explicit strict-less update.  And when no link's channel
// time depends on the cut position the whole program has a closed form (pp_dp_flat.h).  Which
// of the three applies depends on the data, which the host cannot see without synchronising:
// the pack kernel leaves what is needed to tell in the workspace header, and the one kernel
// enqueued after it branches on that.
#include "pp_common.h"
#include "pp_dp_band.h"
#include "pp_dp_band_table.h"
#include "pp_dp_generic.h"
#include "pp_dp_rows.h"
#include "pp_dp_tile.h"
#include "pp_share.h"

// ---------------------------------------------------------------- pack

struct pack_args {
    int L, D, S, K, nt;
    long long N;
    size_t total;  // D*D*L
    const long long *PF, *PB, *XF, *XB;
    pp_ws_header *hdr;
    int *p32, *x32, *xkt, *xct, *ord;  // ord != NULL: write all D! orderings in lexicographic order
    long long *bfl;                    // [S][L+1] partition DP without channel costs
    int pack;                          // 0: the tables of the links are left to k_share_hash (pp_share.hip)
    band_table_args band;
};

// x32[link*L + k] = XF + XB at cut position k (k layers before the cut), k = 1..L-1; entry 0
// is 0.  Returns this thread's largest entry; clears `flat` if an entry differs from the one
// at the previous cut position of the same link.
__device__ unsigned long long pack_x(const pack_args &a, size_t first, size_t stride, bool &flat) {
    unsigned long long m = 0;
    for (size_t i = first; i < a.total; i += stride) {
        int k = a.total <= 0xffffffffu ? (int)((unsigned)i % (unsigned)a.L) : (int)(i % (size_t)a.L);
        long long x = 0;
        if (k >= 1) x = a.XF[i - 1] + a.XB[i - 1];
        if (k >= 2) flat &= (x == a.XF[i - 2] + a.XB[i - 2]);
        a.x32[i] = (int)x;
        unsigned long long ux = x < 0 ? ~0ull : (unsigned long long)x;
        m = ux > m ? ux : m;
    }
    return m;
}

// Tile layout of the same table as keys, for the register-tiled kernel:
// xkt[(link*8 + b)*nt + j] = (x << K) | k for k = 8j + b, infinite for k == 0 or k >= L.
__device__ void pack_xkt(const pack_args &a, unsigned first, unsigned stride) {
    if (!a.nt) return;
    const unsigned per_link = 8u * a.nt, n = (unsigned)a.D * a.D * per_link;  // D*D*128 < 2^32
    for (unsigned i = first; i < n; i += stride) {
        unsigned link = i / per_link;
        int r = (int)(i - link * per_link);
        int b = r / a.nt, j = r - b * a.nt, k = 8 * j + b;
        int key = PP_INF32;
        if (k >= 1 && k < a.L) {
            long long x = a.XF[(size_t)link * a.L + k - 1] + a.XB[(size_t)link * a.L + k - 1];
            key = (int)(((unsigned)x << a.K) | (unsigned)k);
        }
        a.xkt[i] = key;
    }
}

// The same keys once more in the layout of the cells a lane holds after a row's reduction
// (lane (a, b) holds the cells l = 8 (h H + r) + a + 1, h = b / 4, r = 0..H-1, H = ceil(nt / 2)):
// xct[((link*8 + a)*2 + h)*H + r] = (x << K) | l, infinite for l >= L or a tile beyond nt.
__device__ void pack_xct(const pack_args &a, unsigned first, unsigned stride) {
    if (!a.nt) return;
    const unsigned H = (unsigned)(a.nt + 1) / 2, per_link = 16u * H, n = (unsigned)a.D * a.D * per_link;
    for (unsigned i = first; i < n; i += stride) {
        unsigned link = i / per_link, r0 = i - link * per_link;
        unsigned la = r0 / (2 * H), h = (r0 / H) & 1u, r = r0 % H;
        int tile = (int)(h * H + r), l = 8 * tile + (int)la + 1;
        int key = PP_INF32;
        if (tile < a.nt && l < a.L) {
            long long x = a.XF[(size_t)link * a.L + l - 1] + a.XB[(size_t)link * a.L + l - 1];
            key = (int)(((unsigned)x << a.K) | (unsigned)l);
        }
        a.xct[i] = key;
    }
}

// Row c of the explicit list = the ordering of lexicographic rank c.  Its factorial-number
// digits come out least significant first by dividing by 1, 2, 3, ...: digit n (counted from
// the front) = (c / (D-1-n)!) mod (D-n); digit n selects the digit-th smallest unused device.
// 32-bit arithmetic when D! fits (D <= 12).
__device__ void unrank_rows(const pack_args &a, long long first, long long stride) {
    const int D = a.D;
    for (long long c = first; c < a.N; c += stride) {
        unsigned long long digits = 0;  // 5 bits per digit: digits 0..11 here, 12..19 in digits_hi
        unsigned long long digits_hi = 0;
        if (D <= 12) {
            unsigned rem = (unsigned)c;
#pragma unroll
            for (int i = 1; i <= 12; ++i) {  // i = D - n; unrolled: divisions by constants
                if (i > D) break;
                unsigned q = rem / (unsigned)i;
                unsigned long long dg = rem - q * (unsigned)i;
                rem = q;
                digits |= dg << (5 * (D - i));
            }
        } else {
            unsigned long long rem = (unsigned long long)c;
            for (int i = 1; i <= D; ++i) {
                unsigned long long q = rem / (unsigned long long)i;
                unsigned long long dg = rem - q * (unsigned long long)i;
                rem = q;
                int n = D - i;
                if (n < 12) digits |= dg << (5 * n);
                else digits_hi |= dg << (5 * (n - 12));
            }
        }
        unsigned used = 0;
        int row[4];
        const bool vec = (D & 3) == 0;  // rows are 16-byte aligned pieces: store four devices at a time
        for (int n = 0; n < D; ++n) {
            int digit = (int)(((n < 12 ? digits >> (5 * n) : digits_hi >> (5 * (n - 12)))) & 31);
            // digit-th zero bit of `used`
            unsigned freeb = ~used;
            for (int k = 0; k < digit; ++k) freeb &= freeb - 1;
            int dev = __builtin_ctz(freeb);
            used |= 1u << dev;
            if (vec) {
                row[n & 3] = dev;
                if ((n & 3) == 3) *(int4 *)(a.ord + c * D + n - 3) = make_int4(row[0], row[1], row[2], row[3]);
            } else {
                a.ord[c * D + n] = dev;
            }
        }
    }
}

// The partition DP with every channel cost taken as zero, which does not depend on the
// candidate: B[0][l] = P[l], B[n][l] = min_{n<=k<l} max(B[n-1][k], P[l] - P[k]) (infinite for
// l <= n), and A[n][l] = the lowest minimising k.  pp_dp_flat.h builds every candidate's plan
// from these two tables when no link's channel time depends on the cut position.  Rows are
// non-decreasing in l and P[l] - P[k] falls as k grows, so a cell is decided at the first
// split k* where the two cross (binary search): left of it the difference is the larger term,
// from it on the previous row.  If the difference just left of the crossing is no larger than
// the row value at it, the minimum sits there, at the lowest split with that same prefix sum
// (zero-length layers make equal neighbours); otherwise at k*.
// One workgroup; sh holds P and two rows.  a.bfl: B [S][L+1] int64, then A [S][L+1] int32.
__device__ void flat_table(const pack_args &a, long long *sh) {
    const int L = a.L, S = a.S, tid = threadIdx.x;
    // The tables are read only when no link's channel time depends on the cut position.  If
    // some link's times at the first two cut positions already differ, that is not so (the
    // pack blocks will find the same), and the work below can be left out.  Only for long
    // models: for L <= 128 the table is cheap and this launch is on the path of a step of a few
    // tens of microseconds, where the test's own barriers cost more than it can save.
    // (this thread's first entry of P is requested here, so that it travels with the loads of the test)
    const long long p_first = tid <= L ? a.PF[tid] + a.PB[tid] : 0;
    if (L > PP_TILE_MAX_L) {
        __shared__ int s_differs;
        if (tid == 0) s_differs = 0;
        __syncthreads();
        bool differs = false;
        for (int link = tid; link < a.D * a.D; link += 256) {
            if (link / a.D == link % a.D) continue;
            const size_t at = (size_t)link * L;
            differs |= a.XF[at] + a.XB[at] != a.XF[at + 1] + a.XB[at + 1];
        }
        if (differs) s_differs = 1;
        __syncthreads();
        if (s_differs) return;
    }
    long long *P = sh, *cur = sh + (L + 1), *nxt = cur + (L + 1);
    int *A = (int *)(a.bfl + (size_t)S * (L + 1));
    for (int l = tid; l <= L; l += 256) {
        const long long p = l == tid ? p_first : a.PF[l] + a.PB[l];
        P[l] = p;
        cur[l] = p;
        a.bfl[l] = p;
        A[l] = 0;
    }
    __syncthreads();
    for (int n = 1; n < S; ++n) {
        for (int l = tid; l <= L; l += 256) {
            long long best = PP_INF64;
            int arg = 0;
            if (l >= n + 1) {
                const long long Pl = P[l];
                int lo = n, hi = l;  // first split k in [n, l) with row[k] >= P[l] - P[k], or l
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (cur[mid] >= Pl - P[mid]) hi = mid;
                    else lo = mid + 1;
                }
                arg = lo;
                if (lo <= l - 1) best = cur[lo];
                if (lo - 1 >= n) {
                    const long long d = Pl - P[lo - 1];
                    if (d <= best) {
                        best = d;
                        int k = lo - 1;
                        while (k > n && P[k - 1] == P[k]) --k;
                        arg = k;
                    }
                }
            }
            nxt[l] = best;
            a.bfl[(size_t)n * (L + 1) + l] = best;
            A[(size_t)n * (L + 1) + l] = arg;
        }
        // The next row reads this one from LDS only, so the barrier waits for the LDS writes and
        // lets the stores to global memory drain behind it (__syncthreads would wait for them
        // too: a trip to memory per row).
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        long long *t = cur; cur = nxt; nxt = t;
    }
}

// Blocks 0..PP_PACK_BLOCKS-1 pack a slice of the tables each (where candidates may share a DP, L > 128, the kernel
// that reads every link's times to tell them apart does it: 55 -> 16 us at L = 400, D = 64) and record the largest time of
// their slice in the header (no atomics, nothing to initialise); further blocks, if any, write
// the explicit list of all D! orderings.  Block PP_PACK_BLOCKS builds the channel-free DP table, the one
// after it the bands.
__global__ __launch_bounds__(256) void k_prep(pack_args a) {
    extern __shared__ __align__(16) long long dyn[];
    __shared__ unsigned long long sh[4];
    __shared__ int shf[4];
    const int tid = threadIdx.x;
    if (blockIdx.x < PP_PACK_BLOCKS) {
        const unsigned first = blockIdx.x * 256 + tid, stride = PP_PACK_BLOCKS * 256;
        unsigned long long m = 0;
        if (blockIdx.x == 0) {
            // P as int32, padded with P[L] up to a whole tile
            for (int l = tid; l <= a.L + 16; l += 256) {
                int q = l < a.L ? l : a.L;
                a.p32[l] = (int)(a.PF[q] + a.PB[q]);
            }
            long long pl = a.PF[a.L] + a.PB[a.L];
            m = pl < 0 ? ~0ull : (unsigned long long)pl;
            if (tid < 64) {
                if (tid == 0) a.hdr->free_valid = 0;
                auto &w = a.hdr->work[tid];
                w.pairs = w.rows = w.band_pairs = w.band_rows = w.free_rows = 0;
            }
        }
        bool flat = true;
        if (a.pack) {
            const unsigned long long mx = pack_x(a, first, stride, flat);
            m = mx > m ? mx : m;
            pack_xkt(a, first, stride);
            pack_xct(a, first, stride);
        }
        for (int off = 32; off; off >>= 1) {
            unsigned long long o = __shfl_xor(m, off);
            m = o > m ? o : m;
        }
        const int wflat = __ballot(!flat) == 0;
        if ((tid & 63) == 0) { sh[tid >> 6] = m; shf[tid >> 6] = wflat; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < 4; ++w) m = sh[w] > m ? sh[w] : m;
            a.hdr->pmax[blockIdx.x] = m;
            a.hdr->flat[blockIdx.x] = (unsigned)(shf[0] & shf[1] & shf[2] & shf[3]);
        }
    } else if (blockIdx.x == PP_PACK_BLOCKS) {
        flat_table(a, dyn);
    } else if (blockIdx.x == PP_PACK_BLOCKS + 1) {
        if (a.band.table) band_table(a.band, (unsigned char *)dyn);
    } else {
        unrank_rows(a, (long long)(blockIdx.x - PP_PACK_BLOCKS - 2) * 256 + tid,
                    (long long)(gridDim.x - PP_PACK_BLOCKS - 2) * 256);
    }
}

// 8-cell tiles per row of the register-tiled kernel where it does the DP, 0 where another kernel does.
//
// For 88 < L <= 128 the pairs the tiled kernel evaluates (two waves per SIMD by its registers, fewer by LDS)
// stand against the latency of the row kernel's searches, which more resident waves hide.  Measured for
// S = 2 .. 64 with 50 000 sampled orderings, DP alone, tiled / rows in us: 16 against 8 waves per compute
// unit 189 / 142 (L = 89, S = 8), 206 / 145 (L = 128, S = 8); 12 against 8: 288 / 236 (L = 97, S = 11);
// 8 against 6: 846 / 473 (L = 128, S = 16), but 480 / 432 and, with links that bind everywhere, 479 / 544
// (30 000, L = 97, S = 24); 8 against 8: 332 / 376 (L = 89, S = 13), 289 / 349 (L = 112, S = 12).
// Short lists leave SIMDs without a second wave: 1000 candidates 18 / 24 (L = 89, S = 8), 4000 26 / 28, 8000
// 46 / 38; L = 128: 4000 30 / 26; one wave of the tiled kernel per SIMD: 2000 56 / 39 (L = 128, S = 16).
static int pp_dp_tiles(int L, int D, int S, int64_t N, const pp_ws_layout &lay) {
    if (!lay.nt || L <= PP_PAIRS_MAX_L) return lay.nt;
    size_t lds;
    const int wpb = pp_dp_tile_shape(L, D, S, lay.nt, &lds);
    lds = (lds + sizeof(dp_generic_small) + 1279) / 1280 * 1280;
    int tiled = (int)(160 * 1024 / lds) * wpb;
    tiled = tiled < 8 ? tiled : 8;
    // (with the room the stage-count search needs, so that preparation and search agree)
    const int rows = pp_dp_rows_shape(L, D, S, 1).waves_per_cu;
    const int least = tiled <= 6 ? 2048 : (L > 104 ? 4096 : 6144);
    return N >= least && (L > 104 ? rows > tiled : 3 * rows > 4 * tiled) ? 0 : lay.nt;
}

// How the bands of pp_dp_band.h are used: where whole rows of all candidates take so long that looking for plans
// that need none costs little if there are none.  Looking for the channel-free plan costs next to nothing where links
// bind so often that the table's block finds nothing to be had (BAND_SAMPLE); for the recursion over the bands' cells
// see band_cells.  (Below: whole calls of pp_partition_dp in us, without; with bands
// and links that never bind; with bands and links that bind nearly everywhere.)
//
// L > 128: the preparation of shared DPs looks for the channel-free plan of every list of a wave and more: 64
// candidates 61; 44; 64 (L = 150, S = 8), 116; 78; 140 (150, 32), 394; 94; 473 against 469 without (1024, 32).  The
// worst are short lists with links that seldom bind, but where it matters: 76 -> 91 (300, 8), 432 -> 508 (400, 64);
// for L <= 128 56 -> 65 (3000 candidates, 128, 16), 64 -> 72 (20 000, 128, 8).
// With plans of every stage count the table takes 0.11 S^2 us and more: 119; 288; 143 against 140 (150, 32), but 397;
// 227; 476 against 472 (1024, 32).
//
// L <= 128: the row kernel, and the tiled one of few tiles, finish the candidates with the channel-free plan themselves
// where the links' words fit the LDS (band_link_bytes): 33; 23; 34 (6000 candidates, L = 128, S = 8), 50; 24; 53 (all 8!
// orderings), 69; 31; 71 (10 000, 97, 11), 77; 24; 81 (60 000, 40, 8); all 7! orderings 22.5; 21.5; 23.8 are too few.
// Otherwise in launches of their own: 63; 31; 68 (8!, L = 88), 121; 29; 127 (40 000, 88, 8), 164; 58; 173 (8000, 60,
// 33), 81; 29; 87 (40 000, 100, 6), but 48; 28; 52 (10 000, 88, 8) and 22; 26; 26 (2600).  (With that in it, the tiled
// kernel of more tiles has a wave per SIMD less: 175 -> 261 at 300 000, L = 64, S = 4, with links that bind.)
static double band_rows_work(int L, int S, int64_t N, bool lex) {
    return (double)N * (S - 1) * L / (lex ? 3 : 1);  // (a list of all orderings shares two rows in three)
}

// About what whole rows take, in us: for L > 128 a wave's trips from row to row or the cells of all; else the cells, and
// with the tiled kernel the latency of a row, which the waves of a compute unit that its LDS has room for share (236 ps a
// row of 32 cells with 12 waves, 481 of 60 with 6, 614 of 77 with 5, 389 of 88 with 12).
static double band_whole_us(int L, int D, int S, int64_t N, bool lex, const pp_ws_layout &lay) {
    const double work = band_rows_work(L, S, N, lex);
    if (!lay.nt) {
        const double trips = (S - 1) * (1.5 + 0.01 * L), cells = 4e-6 * work;
        return trips > cells ? trips : cells;
    }
    if (!pp_dp_tiles(L, D, S, N, lay)) return 4e-6 * work;
    size_t lds;
    const int wpb = pp_dp_tile_shape(L, D, S, lay.nt, &lds), waves = (int)(160 * 1024 / lds) * wpb;
    return work / L * (4e-6 * L + 1.6e-3 / (waves > 1 ? waves : 1));
}

// How far N candidates are from being enough for the recursion over the bands' cells, which takes a wave some 80 + S us
// (L > 128) or 40 + 4 S whatever comes of it, S / 2 times as much for plans of every stage count: 0 not enough; 1 if
// the table's block finds that it probably ends most of them (a third of the time whole rows take); 2 in any case (a tenth).
// Where it ends them: 3780 -> 316 (200 000 candidates, L = 300, S = 16), 1410 -> 626 (8000, 1024, 32), 1112 -> 542 (270 000,
// 97, 11), 1800 -> 76 (100 000, 77, 30).  Where it does not: 668 -> 734 (270 000, 128, 8), 958 -> 1029 (40 000, 1024, 8), and
// what the two rules keep it from: 910 -> 1067 (2000, 1024, 64), 880 -> 970 (40 000, 300, 16), 64 -> 135 (2000, 150, 8),
// 54 -> 110 (3000, 128, 16), 60 -> 241 (300, 150, 8, every stage count).  A caller's list in sorted order, whose neighbours
// share rows, takes less than the rule thinks, and pays the most: 257 -> 363 (500 000 sorted orderings of 8 devices, L = 128,
// one of them with links that bind at every cut).
static int band_cells(int L, int D, int S, int64_t N, int stages, bool lex, const pp_ws_layout &lay) {
    const double price = (lay.nt ? 40 + 4 * S : 80 + S) * (stages ? S / 2 + 1 : 1);
    const double whole = band_whole_us(L, D, S, N, lex, lay);
    return whole >= 10 * price ? 2 : whole >= 3 * price ? 1 : 0;
}

static int band_use(int L, int D, int S, int64_t N, int stages, bool lex, const pp_ws_layout &lay) {
    if (!lay.band || D > 64) return BAND_USE_NOT;
    const double work = band_rows_work(L, S, N, lex);
    if (!lay.nt) {
        if (!lay.sh_table) return BAND_USE_NOT;
        int waves = 1;
        band_table_lds(L, S, stages, waves);
        return !stages || band_whole_us(L, D, S, N, lex, lay) >= (double)S * S / waves ? BAND_USE_INSIDE : BAND_USE_NOT;
    }
    const bool room = (size_t)band_link_words(D, S, stages) * 8 + (size_t)N / 8 + 8 <= (size_t)N * 8;  // (in lay.left)
    const bool inside = pp_dp_tiles(L, D, S, N, lay) <= DPT_INSIDE_NT && band_link_bytes(D, S, stages) != 0;
    if (room && band_cells(L, D, S, N, stages, lex, lay)) return BAND_USE_ALONE;
    if (inside) return work >= 3e6 ? BAND_USE_INSIDE : BAND_USE_NOT;
    return room && work >= 8e6 ? BAND_USE_ALONE : BAND_USE_NOT;
}

int pp_launch_pack(int L, int D, int S, int64_t N, const int64_t *PF, const int64_t *PB,
                   const int64_t *XF, const int64_t *XB, const int32_t *orderings, int stages, void *ws,
                   const pp_ws_layout &lay, const int32_t **ord, hipStream_t st) {
    char *base = (char *)ws;
    pack_args a;
    a.L = L; a.D = D; a.S = S; a.K = pp_index_bits(L); a.nt = pp_dp_tiles(L, D, S, N, lay); a.N = N;
    a.total = (size_t)D * D * L;
    a.PF = (const long long *)PF; a.PB = (const long long *)PB;
    a.XF = (const long long *)XF; a.XB = (const long long *)XB;
    a.hdr = (pp_ws_header *)(base + lay.hdr);
    a.p32 = (int *)(base + lay.p32);
    a.x32 = (int *)(base + lay.x32);
    a.xkt = (int *)(base + lay.xkt);
    a.xct = (int *)(base + lay.xct);
    a.bfl = (long long *)(base + lay.bfl);
    a.ord = orderings ? NULL : (int *)(base + lay.ord);
    *ord = orderings ? orderings : (const int32_t *)(base + lay.ord);
    a.pack = !lay.sh_table;
    band_table_args &t = a.band;
    t.L = L; t.D = D; t.S = S; t.K = a.K;
    t.PF = a.PF; t.PB = a.PB; t.XF = a.XF; t.XB = a.XB;
    t.table = band_use(L, D, S, N, stages, orderings == NULL, lay) ? (int *)(base + lay.band) : NULL;
    t.waves = 1;
    t.stages = stages;
    t.cells = band_cells(L, D, S, N, stages, orderings == NULL, lay);
    t.fit_limit = (1ull << (31 - a.K)) - 1;
    int grid = PP_PACK_BLOCKS + 2;
    size_t lds = (size_t)3 * (L + 1) * 8;
    const size_t band_lds = band_table_lds(L, S, stages, t.waves);
    if (t.table && lds < band_lds) lds = band_lds;
    if (a.ord) grid += (int)((N + 255) / 256 < 1024 ? (N + 255) / 256 : 1024);
    hipLaunchKernelGGL(k_prep, dim3(grid), dim3(256), lds, st, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}

// ---------------------------------------------------------------- launch policy

// Consecutive candidates one wave of the tiled kernel walks.
//
// Caller's list: split it evenly over the resident waves.  All D! orderings in
// lexicographic order: consecutive candidates share ordering prefixes and with them DP rows,
// so a wave that walks c candidates computes about c * r + (D - 2 - r) full rows, where
// r = sum_{m=1}^{D-2} 1/m! is the average number of rows that change from one ordering to
// the next; a chunk of k! candidates aligned to a multiple of k! shares its first D-k
// devices and needs exactly (D-k-1) + sum_{n>=D-k} k!/(D-1-n)! rows.  The kernel is bound by
// instruction issue, so a SIMD that holds w waves takes about w times as long as one that
// holds a single wave would at full rate, except that a lone wave cannot hide its own LDS
// and issue latencies and runs about 1.4 times slower per row.  Pick the size that minimises
// (waves on the busiest SIMD) x (rows per wave) under that model.
static long long choose_chunk(int64_t N, int D, bool lex, long long simds, int waves_per_simd) {
    const long long slots = simds * waves_per_simd;
    const long long even = (long long)((N + slots - 1) / slots);
    if (!lex || D < 3) return even;
    double r = 0, term = 1;
    for (int m = 1; m <= D - 2; ++m) { term /= m; r += term; }
    auto cost = [&](long long c, double rows) {
        long long nwaves = (long long)((N + c - 1) / c);
        long long per_simd = (nwaves + simds - 1) / simds;
        if (per_simd > waves_per_simd)  // later waves start as earlier ones finish
            return rows * (double)nwaves / (double)simds;
        return rows * (per_simd <= 1 ? 1.4 : (double)per_simd);
    };
    long long best = even;
    double best_cost = cost(even, even * r + (D - 2 - r) + 0.1 * even);
    long long f = 1;
    for (int k = 1; k < D; ++k) {
        f *= k;
        if (f > N) break;
        double rows = 0.1 * (double)f;  // last row: one cell per candidate
        for (int n = 1; n <= D - 2; ++n) {
            double nodes = 1;  // row n is shared by the whole chunk when n <= D-k-1
            if (n >= D - k) {
                nodes = (double)f;
                for (int q = 2; q <= D - 1 - n; ++q) nodes /= q;
            }
            rows += nodes;
        }
        double c = cost(f, rows);
        if (c < best_cost) { best_cost = c; best = f; }
    }
    return best;
}

pp_free_plans pp_free_of(void *ws, const pp_ws_layout &lay, int S) {
    if (!lay.fx) return {NULL, NULL, NULL};
    return {(const unsigned long long *)((char *)ws + lay.fbits), (const long long *)((char *)ws + lay.fleast),
            (const int *)((char *)ws + lay.band) + band_plan_at(S, S)};
}

int pp_launch_dp(int L, int D, int S, int64_t N, const int64_t *PF, const int64_t *PB,
                 const int64_t *XF, const int64_t *XB, const int32_t *lex_ord,
                 const int32_t *user_ord, int stages, int defer_mmax, int keep_list,
                 pp_sched_info *sched, int64_t *C_out, int32_t *bounds_out, void *ws, const pp_ws_layout &lay,
                 int32_t *status, hipStream_t st) {
    if (keep_list && !lay.sh_table) return PP_ERR_INVALID_ARG;
    char *base = (char *)ws;
    dp_args a;
    a.stages = stages;
    a.L = L; a.D = D; a.S = S; a.K = pp_index_bits(L); a.N = N;
    a.fit_limit = (1ull << (31 - a.K)) - 1;
    a.PF = (const long long *)PF; a.PB = (const long long *)PB;
    a.XF = (const long long *)XF; a.XB = (const long long *)XB;
    a.ord = lex_ord ? lex_ord : user_ord;
    a.validate = user_ord != NULL;
    a.hdr = (pp_ws_header *)(base + lay.hdr);
    a.p32 = (const int *)(base + lay.p32);
    a.x32 = (const int *)(base + lay.x32);
    a.arg = (unsigned short *)(base + lay.arg);
    a.C_out = (long long *)C_out;
    a.bounds_out = bounds_out;
    a.status = status;
    a.nblocks = lay.slots;
    a.bfl = (const long long *)(base + lay.bfl);
    a.defer_mmax = defer_mmax;
    const int use = band_use(L, D, S, N, stages, lex_ord != NULL, lay);
    a.band = use ? (const int *)(base + lay.band) : NULL;
    // (representatives are fewer than the candidates the rule has looked at)
    a.band_all = band_cells(L, D, S, N, stages, lex_ord != NULL, lay) ? 0 : N + 1;
    if (!a.band_all && lay.sh_table)
        for (a.band_all = 64; a.band_all < N && !band_cells(L, D, S, a.band_all, stages, false, lay);) a.band_all *= 2;
    a.left = NULL;
    a.fx = NULL;
    a.fbits = NULL;
    a.fT = a.fleast = NULL;
    a.f_nM = 0;
    // (Bands of a launch of their own: k_dp_rows looks at the candidates itself.  L > 128: not where candidates share their DP
    // whatever the links are, because k_band_free would find that and leave: 3 us of 67 to 105 for 2 or 3 of 12 to 30 devices.
    // With more stages only the device knows; where they don't share, it saves 1 to 8 us of lists as short as 64.)
    const bool shared = lay.sh_table && share_table_size((unsigned)(D * D), S) != 0;
    if (sched && sched->nM <= PP_FREE_COUNTS && !stages && lay.fx && (use == BAND_USE_ALONE || (a.band && lay.sh_table && !shared))) {
        sched->looked = true;
        a.fx = (int2 *)(base + lay.fx);
        a.fbits = (unsigned long long *)(base + lay.fbits);
        a.fT = (long long *)sched->T;
        a.fleast = (long long *)(base + lay.fleast);
        a.f_nM = sched->nM;
        for (int q = 0; q < PP_FREE_COUNTS; ++q) a.f_Ms[q] = q < sched->nM ? sched->Ms[q] : 1;
    }

    int cus = 256;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    // Priority levels of the waves that share a SIMD end when a tenth, a quarter and half of the chunk
    // are left: they drift apart while they are on the same level and are pulled together at each
    // boundary, so the levels get shorter towards the end (the tiled kernel, L = 128, all 8! orderings,
    // against equal quarters: 65.8 against 67.1 us).
    auto levels = [](long long chunk, int (&left)[3]) {
        const long long frac[3] = {10, 4, 2};
        for (int k = 0; k < 3; ++k) {
            const long long v = chunk / frac[k];
            left[k] = (int)(v > 0x3fffffff ? 0x3fffffff : v);
        }
    };
    const int nt = pp_dp_tiles(L, D, S, N, lay);
    if (use == BAND_USE_ALONE) {
        // (in lay.left; with the links' times, where these are)
        unsigned long long *left = (unsigned long long *)(base + lay.left), *words = left;
        if (a.fx) words = (unsigned long long *)a.fx;
        else left += band_link_words(D, S, stages);
        a.left = left;
        const int rc = pp_launch_dp_band_alone(a, words, left, st);
        if (rc) return rc;
    }
    if (lay.nt && !nt) {
        dp_rows_args t;
        t.L = L; t.D = D; t.S = S; t.K = a.K; t.N = N;
        t.validate = a.validate;
        const dpr_shape sh = pp_dp_rows_shape(L, D, S, stages);
        if (!sh.wpb) return PP_ERR_INVALID_ARG;  // cannot happen for S <= 64
        // the list split evenly over the resident waves, also where neighbours share rows: the kernel
        // is bound by latency, and with all 8! orderings of L = 128 runs of 4! (two waves per SIMD)
        // took 110 us for the whole search, runs of 10 (four) 78 us
        t.chunk = (N + (long long)cus * sh.waves_per_cu - 1) / ((long long)cus * sh.waves_per_cu);
        levels(t.chunk, t.prio_left);
        const long long nchunks = (N + t.chunk - 1) / t.chunk;
        const int grid = (int)((nchunks + sh.wpb - 1) / sh.wpb);
        if (a.nblocks > grid) a.nblocks = grid;
        t.g = a;
        return pp_launch_dp_rows(t, grid, sh, st);
    }
    if (nt) {
        // register-tiled kernel, one wave per candidate (falls back to the generic
        // int64 body inside the same launch when the times do not fit 32-bit keys)
        dp_tile_args t;
        t.L = L; t.D = D; t.S = S; t.K = a.K; t.N = N;
        t.validate = a.validate;
        t.xkt = (const int *)(base + lay.xkt);
        t.xct = (const int *)(base + lay.xct);
        size_t lds;
        const int wpb = pp_dp_tile_shape(L, D, S, nt, &lds);
        if (!wpb) return PP_ERR_INVALID_ARG;  // cannot happen for S <= 64
        const int waves_per_simd = nt >= 14 ? 2 : (nt >= 12 ? 3 : 4);
        t.chunk = choose_chunk(N, D, lex_ord != NULL, (long long)cus * 4, waves_per_simd);
        levels(t.chunk, t.prio_left);
        const long long nchunks = (N + t.chunk - 1) / t.chunk;
        const int grid = (int)((nchunks + wpb - 1) / wpb);
        if (a.nblocks > grid) a.nblocks = grid;
        t.g = a;
        return pp_launch_dp_tile(t, nt, grid, wpb, st);
    }
    // L > 128: one persistent wave per candidate slot
    long long waves = lay.slots < N ? lay.slots : N;
    if (!lay.sh_table) return pp_launch_dp_big(a, (int)waves, cus, NULL, st);
    // candidates whose links have the same channel times share one DP: the kernel walks the
    // representatives the preparation finds, and their results are copied to the others
    const int run_waves = pp_dp_big_run_waves(pp_dp_big_waves(L, D, S, (int)waves, cus), S, lay.sh_row_slots);
    int rc = pp_launch_share_prepare(a, run_waves, ws, lay, st);
    if (rc) return rc;
    pp_share_list list;
    list.reps = (const int *)(base + lay.sh_reps);
    list.pend = (const int *)(base + lay.left);
    list.keys = (const int *)(base + lay.sh_keys);
    list.start = (const int *)(base + lay.sh_start);
    list.rows = (int *)(base + lay.sh_rows);
    list.row_slots = lay.sh_row_slots;
    rc = pp_launch_dp_big(a, (int)waves, cus, &list, st);
    if (rc || keep_list) return rc;
    return pp_launch_share_scatter(N, stages ? S : 1, stages ? S * (S + 1) / 2 : S, 0, 1, C_out,
                                   bounds_out, NULL, ws, lay, st);
}
