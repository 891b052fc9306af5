// One partition DP for all candidates that are the same problem.
//
// Row n of the recursion for W(l, xi, r, i) (Sec. IV-B with one replica per stage) sees a
// candidate's devices only through X_n[k], the time link (o[n-1], o[n]) needs for the
// activations at cut position k.  Real clusters have few distinct bandwidths (Sec. III-A: PCIe
// or NVLink inside a server, RDMA or TCP between servers; the testbeds of Sec. V-A have one of
// each), so many links carry the same row X[.], and two candidates whose links have equal rows
// position by position get the same table, bottleneck and plan.  This file finds those groups
// on the device:
//   1. k_share_hash     a hash of every link's forward and backward row (one wave per link), the link's
//                       times packed for the DP, and the table of representatives set to "none";
//   2. k_share_classes  link i joins the class of the lowest link with the same hash whose rows
//                       are equal entry by entry (one wave per link), and the classes are counted;
//   3. k_share_keys     classes numbered 0..nc-1; a candidate's key is its sequence of S-1
//                       class numbers read as a number in base nc (first link most
//                       significant), and the lowest candidate of every key is kept with an
//                       atomic min (only if nc^(S-1) fits the table);
//   4. k_share_count, k_share_reps   the table compacted, in the order of the keys, into the
//                       list of representatives;
//   5. k_dp_band        (pp_dp_band.hip) finishes the representatives whose few best cells suffice;
//   6. k_share_cost, k_share_bounds  the others cut into runs of about equal work, one per wave
//                       of the DP kernel.
// The DP kernel walks the list - neighbours in it share their first links and with them the
// first rows of the table - and k_share_scatter hands every representative's results to the
// candidates of its key.  Candidates with a bad ordering are representatives of themselves
// (kept after the sorted ones), so the DP kernel reports them as it always does.
//
// When the keys do not fit the table (every link its own class) there is still something to
// share: row n depends on the first n + 1 devices only, and a long sampled list holds each
// choice of the first few devices many times.  What the bands leave of the candidates is then
// sorted by the first k devices (D^k <= table entries; a counting sort: histogram in k_dp_band
// before the keys, bucket offsets in k_share_count / k_share_reps, placement in k_dp_band after
// them), and the DP kernel reuses the first k - 1 rows between neighbours.  All decisions are taken
// on the device.
#include "pp_dp_band.h"
#include "pp_share.h"

struct share_args {
    int L, D, S, validate;
    long long N;
    const long long *XF, *XB;
    int *x32;                   // [D*D*L] XF + XB (entry k: the cut after k layers)
    const int *ord;
    dp_args g;                  // what the bands need of it: the tables
    const int *band;            // the pack kernel's table of the bands, or NULL
    int sort;                   // lists whose keys do not fit are sorted by their first devices
    unsigned long long *links;  // band_links' words
    pp_ws_header *hdr;
    unsigned long long *lhash;  // [D*D]
    int *lrep;                  // [D*D] lowest link with equal rows (-1 on the diagonal)
    int *table;                 // [PP_SHARE_TABLE] lowest candidate of every key
    int *keys;                  // [N] key of every candidate (-1: bad ordering)
    int *reps;                  // [N] representatives (see pp_share_at)
    int *cnt;                   // [PP_SHARE_TABLE / 256] keys in use per 256 table entries
    int *pend;                  // [N] representatives the bands have left
    int *start;                 // [run_waves + 1] first entry of every run of that list
    int run_waves;
    long long first_c, last_c;  // k_share_keys: candidates first_c .. last_c - 1
    // scatter
    int nC, nB, nT, tw, vec;
    long long *C_out, *T_out;
    int *bounds_out;
};

#define SHARE_FILL_BLOCKS 256

// (a finaliser in the style of splitmix64: multiply, fold the high bits down, twice)
__device__ __forceinline__ unsigned long long share_mix(unsigned long long z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void k_share_hash(share_args a) {
    const int nl = a.D * a.D, hash_blocks = (nl + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63;
    if ((int)blockIdx.x >= hash_blocks) {
        // the table of representatives: every key empty
        const int b = blockIdx.x - hash_blocks;
        int4 *t4 = (int4 *)a.table;
        const int4 none = make_int4(SHARE_NONE, SHARE_NONE, SHARE_NONE, SHARE_NONE);
        for (int i = b * 256 + tid; i < PP_SHARE_TABLE / 4; i += SHARE_FILL_BLOCKS * 256) t4[i] = none;
        return;
    }
    if (blockIdx.x == 0 && tid == 0) {
        a.hdr->share_active = 0;
        a.hdr->share_nc = 0;
        a.hdr->share_tsize = 0;
        a.hdr->share_nreps = 0;
        a.hdr->share_nsorted = 0;
        a.hdr->share_nbad = 0;
        a.hdr->share_sorted = 0;
        a.hdr->share_kdev = 0;
        a.hdr->share_nchunks = 0;
        a.hdr->share_npend = 0;
    }
    const int i = blockIdx.x * 4 + (tid >> 6);
    if (i >= nl) return;
    const int u = i / a.D, v = i - u * a.D;
    const long long *xf = a.XF + (size_t)i * a.L, *xb = a.XB + (size_t)i * a.L;
    int *x32 = a.x32 + (size_t)i * a.L;
    unsigned long long h = 0, m = 0;
    bool flat = true;
    const long long first = xf[0] + xb[0];
    // the entries a plan can read: cut positions 1..L-1, stored at 0..L-2
    for (int k = lane; k < a.L - 1; k += 64) {
        const long long f = xf[k], b = xb[k], x = f + b;
        h += share_mix(share_mix((unsigned long long)f + 0x9E3779B97F4A7C15ull * (unsigned)(k + 1)) ^ (unsigned long long)b);
        x32[k + 1] = (int)x;
        flat &= x == first;
        const unsigned long long ux = x < 0 ? ~0ull : (unsigned long long)x;
        m = ux > m ? ux : m;
    }
    for (int off = 32; off; off >>= 1) {
        h += __shfl_xor(h, off);
        const unsigned long long o = __shfl_xor(m, off);
        m = o > m ? o : m;
    }
    const bool all_flat = __ballot(!flat) == 0;
    if (lane == 0) {
        x32[0] = 0;
        a.lhash[i] = u != v ? h : 0;
        atomicMax(&a.hdr->pmax[i & (PP_PACK_BLOCKS - 1)], m);
        if (!all_flat) a.hdr->flat[i & (PP_PACK_BLOCKS - 1)] = 0;  // (set everywhere by the pack kernel)
    }
}

__global__ __launch_bounds__(256) void k_share_classes(share_args a) {
    const int nl = a.D * a.D, D = a.D, L = a.L;
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= nl) return;
    if (i / D == i % D) {
        if (lane == 0) a.lrep[i] = -1;
        return;
    }
    if (a.band) band_link_wave(a.g, a.band, i, a.links);
    const unsigned long long h = a.lhash[i];
    int rep = i;
    for (int base = 0; base < i && rep == i; base += 64) {
        const int j = base + lane;
        const bool m = j < i && j / D != j % D && a.lhash[j] == h;
        unsigned long long mask = __ballot(m);
        while (mask) {
            const int j0 = base + __builtin_ctzll(mask);
            mask &= mask - 1;
            bool diff = false;
            const long long *xi = a.XF + (size_t)i * L, *xj = a.XF + (size_t)j0 * L;
            const long long *yi = a.XB + (size_t)i * L, *yj = a.XB + (size_t)j0 * L;
            for (int k = lane; k < L - 1; k += 64) diff |= xi[k] != xj[k] || yi[k] != yj[k];
            if (!__ballot(diff)) {
                // the lowest link with these rows: it is its own representative
                rep = j0;
                break;
            }
        }
    }
    if (lane == 0) {
        a.lrep[i] = rep;
        if (rep == i) atomicAdd(&a.hdr->share_nc, 1u);
    }
}

// Candidates of a workgroup and their keys' slots in LDS (k_share_keys, first launch).
#define SHARE_OWN 1024
#define SHARE_SLOT_BITS 11
#define SHARE_SLOTS (1 << SHARE_SLOT_BITS)

// LOOK: the launch for the rest of a list, T = 256 threads (the dynamic LDS holds the class of every link); else a thread
// per candidate of a workgroup, T = SHARE_OWN.  What bounds it: the atomics on the table, and for the rest of a list the
// orderings' bytes (56 MB in 22 us; 28 with one load of a row in flight).
template <bool LOOK>
__global__ __launch_bounds__(LOOK ? 256 : SHARE_OWN) void k_share_keys(share_args a) {
    constexpr int T = LOOK ? 256 : SHARE_OWN;
    extern __shared__ int s_cls[];
    __shared__ int s_cnt[T / 64], s_key[LOOK ? 1 : SHARE_SLOTS], s_low[LOOK ? 1 : SHARE_SLOTS];
    const int nl = a.D * a.D, D = a.D, S = a.S, tid = threadIdx.x;
    const unsigned nc = a.hdr->share_nc, tsize = share_table_size(nc, S);
    // otherwise: buckets of the first kdev devices (pp_dp_band.hip)
    int kdev = 0;
    unsigned nbuck = 1;
    if (!tsize && a.sort) nbuck = share_buckets(D, S, kdev);
    if (blockIdx.x == 0 && tid == 0) {
        a.hdr->share_tsize = tsize ? tsize : (kdev ? nbuck : 0);
        a.hdr->share_active = tsize != 0;
        a.hdr->share_sorted = kdev != 0;
        a.hdr->share_kdev = (unsigned)kdev;
    }
    if (!tsize) return;
    // class numbers: the rank of a link's representative among the representatives
    const int per = (nl + T - 1) / T, lo = tid * per < nl ? tid * per : nl, hi = lo + per < nl ? lo + per : nl;
    int cnt = 0;
    for (int i = lo; i < hi; ++i) cnt += a.lrep[i] == i;
    int before = cnt;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(before, off);
        before += (tid & 63) >= off ? o : 0;
    }
    if ((tid & 63) == 63) s_cnt[tid >> 6] = before;
    __syncthreads();
    before -= cnt;
    for (int w = 0; w < tid >> 6; ++w) before += s_cnt[w];
    for (int i = lo; i < hi; ++i)
        if (a.lrep[i] == i) s_cls[i] = before++;
    __syncthreads();
    int mine[(PP_SHARE_MAX_D * PP_SHARE_MAX_D + T - 1) / T];
    for (int i = lo; i < hi; ++i) {
        const int r = a.lrep[i];
        mine[i - lo] = r >= 0 ? s_cls[r] : 0;
    }
    __syncthreads();
    for (int i = lo; i < hi; ++i) s_cls[i] = mine[i - lo];
    __syncthreads();
    const bool vec = (S & 3) == 0 && ((uintptr_t)a.ord & 15) == 0;
    // The first launch takes SHARE_OWN neighbours per workgroup and keeps the lowest of every key in LDS first: a
    // key that many candidates have (3.5 % of sampled orderings of 4 servers of 4 devices never stay on a server)
    // would have their atomics queue on its address.  What it has left can be looked at through the caches by
    // the launch for the rest of the list, and is lower than any candidate there.
    if (!LOOK) {
        for (int i = tid; i < SHARE_SLOTS; i += T) { s_key[i] = -1; s_low[i] = SHARE_NONE; }
        __syncthreads();
    }
    for (long long c = a.first_c + (long long)blockIdx.x * T + tid; c < a.last_c; c += (long long)gridDim.x * T) {
        const int *row = a.ord + c * S;
        unsigned long long used = 0;
        unsigned key = 0;
        bool bad = false;
        int prev = 0;
        auto place = [&](int n, int d) {
            if (a.validate) {
                if (d < 0 || d >= D) { bad = true; d = 0; }
                bad |= (used >> d) & 1;
                used |= 1ull << d;
            }
            if (n) key = key * nc + (unsigned)s_cls[prev * D + d];
            prev = d;
        };
        if (vec) {
            // (a row is S devices of 4 bytes: 16 bytes at a time where rows are so aligned)
            // (four of them in flight)
            for (int n0 = 0; n0 < S; n0 += 16) {
                int4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = *(const int4 *)(row + (n0 + 4 * u < S ? n0 + 4 * u : n0));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int n = n0 + 4 * u;
                    if (n >= S) continue;
                    place(n, v[u].x); place(n + 1, v[u].y); place(n + 2, v[u].z); place(n + 3, v[u].w);
                }
            }
        } else {
            for (int n = 0; n < S; ++n) place(n, row[n]);
        }
        if (bad) {
            a.keys[c] = -1;
            a.reps[a.N - 1 - atomicAdd(&a.hdr->share_nbad, 1u)] = (int)c;
            continue;
        }
        a.keys[c] = (int)key;
        if (LOOK) {
            if (a.table[key] > (int)c) atomicMin(&a.table[key], (int)c);
            continue;
        }
        const int slot = (int)((key * 2654435761u) >> (32 - SHARE_SLOT_BITS));
        const int was = atomicCAS(&s_key[slot], -1, (int)key);
        if (was == -1 || was == (int)key) atomicMin(&s_low[slot], (int)c);
        else atomicMin(&a.table[key], (int)c);  // (another key has the slot)
    }
    if (LOOK) return;
    __syncthreads();
    for (int i = tid; i < SHARE_SLOTS; i += T)
        if (s_key[i] >= 0) atomicMin(&a.table[s_key[i]], s_low[i]);
}

// Keys in use in every block of 256 table entries.
__global__ __launch_bounds__(256) void k_share_count(share_args a) {
    __shared__ int sh[4];
    const unsigned tsize = a.hdr->share_tsize;
    const unsigned key = blockIdx.x * 256u + threadIdx.x;
    if (a.hdr->share_sorted && !a.hdr->share_npend) return;  // (the bands have left none)
    int n;
    if (a.hdr->share_sorted) {
        // candidates in the bucket
        n = key < tsize ? (int)((unsigned)a.table[key] - (unsigned)SHARE_NONE) : 0;
        for (int off = 32; off; off >>= 1) n += __shfl_xor(n, off);
    } else {
        const bool has = key < tsize && a.table[key] != SHARE_NONE;
        n = __builtin_popcountll(__ballot(has));
    }
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) a.cnt[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ __launch_bounds__(256) void k_share_reps(share_args a) {
    __shared__ int sh[4], shw[4];
    const int tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    const unsigned tsize = a.hdr->share_tsize;
    if (blockIdx.x * 256u >= tsize && blockIdx.x) return;
    if (a.hdr->share_sorted && !a.hdr->share_npend) return;
    // keys in use before this block's (block 0: in all blocks, for the header)
    const int upto = blockIdx.x ? (int)blockIdx.x : PP_SHARE_TABLE / 256;
    int sum = 0;
    for (int i = tid; i < upto; i += 256) sum += a.cnt[i];
    for (int off = 32; off; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) sh[wib] = sum;
    __syncthreads();
    const int before = sh[0] + sh[1] + sh[2] + sh[3];
    if (blockIdx.x == 0) {
        if (tid == 0) {
            a.hdr->share_nsorted = (unsigned)before;
            a.hdr->share_nreps = (unsigned)before + a.hdr->share_nbad;
        }
    }
    const int base = blockIdx.x ? before : 0;
    const unsigned key = blockIdx.x * 256u + tid;
    if (a.hdr->share_sorted) {
        // every bucket's first position in the list (k_dp_band hands the positions out)
        const int n = key < tsize ? (int)((unsigned)a.table[key] - (unsigned)SHARE_NONE) : 0;
        int incl = n;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off);
            incl += lane >= off ? o : 0;
        }
        if (lane == 63) shw[wib] = incl;
        __syncthreads();
        int at = base + incl - n;
        for (int w = 0; w < wib; ++w) at += shw[w];
        if (key < tsize) a.table[key] = at;
        return;
    }
    const int c = key < tsize ? a.table[key] : SHARE_NONE;
    const bool has = c != SHARE_NONE;
    const unsigned long long mask = __ballot(has);
    if (lane == 0) shw[wib] = __builtin_popcountll(mask);
    __syncthreads();
    int at = base + __builtin_popcountll(mask & ((1ull << lane) - 1));
    for (int w = 0; w < wib; ++w) at += shw[w];
    if (has) a.reps[at] = c;
}

// Work of representative r of the sorted list when it follows r - 1 in a run: the rows its key
// does not share with its predecessor's (at least the last one), plus one row's worth for what
// a candidate costs besides its rows.  A run's first entry computes all S - 1 rows.
// (One that has ended already costs nothing.)
__device__ __forceinline__ int share_cost(const share_args &a, long long r) {
    const int S = a.S;
    const unsigned key = (unsigned)a.keys[a.reps[r]];
    if (key & SHARE_ENDED) return 0;
    if (r == 0 || S < 3) return S;
    const unsigned prev = (unsigned)a.keys[a.reps[r - 1]] & ~(unsigned)SHARE_ENDED;
    const unsigned nc = a.hdr->share_nc;
    unsigned pw = a.hdr->share_tsize / nc;  // weight of the first digit
    int p = 0;
    for (int n = 1; n < S - 1 && key / pw == prev / pw; ++n) { ++p; pw /= nc; }
    return S - p;
}

// Sum of share_cost over every 256 entries of the sorted list (cnt is free again by now), and in the bits from
// SHARE_LEFT on how many of them are left to the DP kernel.
#define SHARE_LEFT 20
__global__ __launch_bounds__(256) void k_share_cost(share_args a) {
    __shared__ int sh[4];
    if (!a.hdr->share_active) return;
    const long long r = (long long)blockIdx.x * 256 + threadIdx.x;
    int c = r < (long long)a.hdr->share_nsorted ? share_cost(a, r) : 0;
    c |= (c != 0) << SHARE_LEFT;
    for (int off = 32; off; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) a.cnt[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// The representatives that are left, in the order of the list, cut into runs of about total / run_waves work
// each (never less than S + 1, so that the running sum crosses at most one boundary per entry): start[w] = first
// entry of run w.
__global__ __launch_bounds__(256) void k_share_bounds(share_args a) {
    __shared__ long long sh[4], s_excl[256];
    __shared__ int shp[4], sht[4];
    if (!a.hdr->share_active) return;
    const int tid = threadIdx.x, lane = tid & 63, wib = tid >> 6;
    const long long ns = a.hdr->share_nsorted;
    if ((long long)blockIdx.x * 256 >= ns) return;
    // work and entries before this block, and in all
    const int nblk = (int)((ns + 255) / 256), low = (1 << SHARE_LEFT) - 1;
    long long before = 0, total = 0;
    int left_before = 0, left_total = 0;
    for (int i = tid; i < nblk; i += 256) {
        const int v = a.cnt[i] & low, p = a.cnt[i] >> SHARE_LEFT;
        total += v;
        left_total += p;
        before += i < (int)blockIdx.x ? v : 0;
        left_before += i < (int)blockIdx.x ? p : 0;
    }
    for (int off = 32; off; off >>= 1) {
        before += __shfl_xor(before, off); total += __shfl_xor(total, off);
        left_before += __shfl_xor(left_before, off); left_total += __shfl_xor(left_total, off);
    }
    if (lane == 0) { sh[wib] = before; s_excl[wib] = total; shp[wib] = left_before; sht[wib] = left_total; }
    __syncthreads();
    before = sh[0] + sh[1] + sh[2] + sh[3];
    total = s_excl[0] + s_excl[1] + s_excl[2] + s_excl[3];
    left_before = shp[0] + shp[1] + shp[2] + shp[3];
    left_total = sht[0] + sht[1] + sht[2] + sht[3];
    if (!total) return;  // (share_nchunks and share_npend are 0)
    __syncthreads();
    long long quota = (total + a.run_waves - 1) / a.run_waves;
    quota = quota > a.S + 1 ? quota : a.S + 1;
    const long long r = (long long)blockIdx.x * 256 + tid;
    const int c = r < ns ? share_cost(a, r) : 0;
    const unsigned long long left = __ballot(c != 0);
    long long incl = c;
    for (int off = 1; off < 64; off <<= 1) {
        const long long o = __shfl_up(incl, off);
        incl += lane >= off ? o : 0;
    }
    if (lane == 63) { sh[wib] = incl; shp[wib] = __builtin_popcountll(left); }
    __syncthreads();
    long long excl = before + incl - c;
    int at = left_before + __builtin_popcountll(left & ((1ull << lane) - 1));
    for (int w = 0; w < wib; ++w) { excl += sh[w]; at += shp[w]; }
    s_excl[tid] = excl;
    __syncthreads();
    if (r >= ns) return;
    if (c) a.pend[at] = a.reps[r];
    const long long id = excl / quota;
    long long id_prev = -1;
    if (tid) id_prev = s_excl[tid - 1] / quota;
    else if (r) id_prev = (excl - share_cost(a, r - 1)) / quota;
    if (id != id_prev) a.start[id] = at;
    if (r == ns - 1) {
        a.start[id + 1] = left_total;
        a.hdr->share_nchunks = (unsigned)(id + 1);
        a.hdr->share_npend = (unsigned)left_total;
    }
}

// Every candidate that is not the representative of its key takes the representative's
// results.
__global__ __launch_bounds__(256) void k_share_scatter(share_args a) {
    if (!a.hdr->share_active) return;
    for (long long c = (long long)blockIdx.x * 256 + threadIdx.x; c < a.N; c += (long long)gridDim.x * 256) {
        const int key = a.keys[c];
        if (key < 0) continue;
        const long long r = a.table[key & ~SHARE_ENDED];
        if (r == c) continue;
        if (a.nC <= 1 && a.tw == 1 && a.nT <= 4 && !a.nB) {
            // (all loads before the first store: one trip to memory)
            const long long C = a.nC ? a.C_out[r] : 0;
            long long t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] = q < a.nT ? a.T_out[q * a.N + r] : 0;
            if (a.nC) a.C_out[c] = C;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q < a.nT) a.T_out[q * a.N + c] = t[q];
            continue;
        }
        for (int i = 0; i < a.nC; ++i) a.C_out[c * a.nC + i] = a.C_out[r * a.nC + i];
        for (int q = 0; q < a.nT; ++q)
            for (int i = 0; i < a.tw; ++i) a.T_out[(q * a.N + c) * a.tw + i] = a.T_out[(q * a.N + r) * a.tw + i];
        if (a.vec) {
            const int4 *src = (const int4 *)(a.bounds_out + r * a.nB);
            int4 *dst = (int4 *)(a.bounds_out + c * a.nB);
            for (int i = 0; i < a.nB / 4; ++i) dst[i] = src[i];
        } else {
            for (int i = 0; i < a.nB; ++i) a.bounds_out[c * a.nB + i] = a.bounds_out[r * a.nB + i];
        }
    }
}

static share_args share_base(void *ws, const pp_ws_layout &lay) {
    char *base = (char *)ws;
    share_args a = {};
    a.hdr = (pp_ws_header *)(base + lay.hdr);
    a.lhash = (unsigned long long *)(base + lay.sh_hash);
    a.lrep = (int *)(base + lay.sh_rep);
    a.table = (int *)(base + lay.sh_table);
    a.keys = (int *)(base + lay.sh_keys);
    a.reps = (int *)(base + lay.sh_reps);
    a.cnt = (int *)(base + lay.sh_cnt);
    a.start = (int *)(base + lay.sh_start);
    a.pend = (int *)(base + lay.left);
    return a;
}

static long long share_grid(int64_t N) {
    const long long g = (N + 255) / 256;
    return g < 4096 ? g : 4096;
}

int pp_launch_share_prepare(const dp_args &g, int run_waves, void *ws, const pp_ws_layout &lay,
                            hipStream_t st) {
    if (!lay.sh_table || run_waves < 1 || run_waves > PP_DP_SLOTS) return PP_ERR_INVALID_ARG;
    share_args a = share_base(ws, lay);
    const int D = g.D;
    const long long N = g.N;
    a.L = g.L; a.D = D; a.S = g.S; a.N = N; a.validate = g.validate;
    a.XF = g.XF; a.XB = g.XB;
    a.x32 = (int *)((char *)ws + lay.x32);
    a.ord = g.ord;
    a.run_waves = run_waves;
    a.g = g;
    a.band = g.band;
    a.sort = N >= 64;  // (no wave of the DP kernel has two candidates of a shorter list)
    // (the saved rows of 64 waves and more, S - 1 of 1040 bytes and more each, hold 8 (S - 1) bytes per link of up
    // to 64 devices, and are needed later; with g.fx the links' times lie behind the words)
    a.links = (unsigned long long *)((char *)ws + lay.sh_rows);
    const int link_blocks = (D * D + 3) / 4;
    hipLaunchKernelGGL(k_share_hash, dim3(link_blocks + SHARE_FILL_BLOCKS), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_share_classes, dim3(link_blocks), dim3(256), 0, st, a);
    int rc = a.sort ? pp_launch_dp_band(g, a.band, a.links, a.keys, a.table, a.reps, 1, st) : PP_OK;
    if (rc) return rc;
    // The keys of a long list in two launches, the first sixteenth alone: 10^6 candidates of 15 751 keys 87 us when
    // every candidate looks past the caches and does its own atomic, 19 + 26 us so (an eighth 30 + 22, a thirty-second 13 + 28).
    const long long first = N > 200000 ? N / 16 : N;
    a.first_c = 0; a.last_c = first;
    hipLaunchKernelGGL(k_share_keys<false>, dim3((unsigned)((first + SHARE_OWN - 1) / SHARE_OWN)), dim3(SHARE_OWN), (size_t)D * D * 4, st, a);
    if (first < N) {
        const long long g = share_grid(N - first);
        a.first_c = first; a.last_c = N;
        hipLaunchKernelGGL(k_share_keys<true>, dim3((unsigned)(g < 2048 ? g : 2048)), dim3(256), (size_t)D * D * 4, st, a);
    }
    hipLaunchKernelGGL(k_share_count, dim3(PP_SHARE_TABLE / 256), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_share_reps, dim3(PP_SHARE_TABLE / 256), dim3(256), 0, st, a);
    rc = a.sort ? pp_launch_dp_band(g, a.band, a.links, a.keys, a.table, a.reps, 0, st) : PP_OK;
    if (rc) return rc;
    hipLaunchKernelGGL(k_share_cost, dim3((unsigned)share_grid(N)), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_share_bounds, dim3((unsigned)share_grid(N)), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}

int pp_launch_share_scatter(int64_t N, int nC, int nB, int nT, int tw, int64_t *C_out,
                            int32_t *bounds_out, int64_t *T_out, void *ws, const pp_ws_layout &lay,
                            hipStream_t st) {
    if (!lay.sh_table) return PP_ERR_INVALID_ARG;
    share_args a = share_base(ws, lay);
    a.N = N; a.nC = nC; a.nB = nB; a.nT = nT; a.tw = tw;
    a.C_out = (long long *)C_out;
    a.T_out = (long long *)T_out;
    a.bounds_out = bounds_out;
    a.vec = nB > 0 && (nB % 4 == 0) && (((uintptr_t)bounds_out & 15) == 0);
    hipLaunchKernelGGL(k_share_scatter, dim3((unsigned)share_grid(N)), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
