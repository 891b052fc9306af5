// pp_schedule_makespan: per-iteration time of a plan under the pipeline execution scheduler
// (Alg. 1, Sec. IV-A), and the candidate arg-min of the SPP listing (Alg. 3).
//
// The scheduler's two phases collapse into a max-plus recurrence.  Its ordering phase moves
// every microbatch one block per sweep, so block j serves microbatch m = t - j + 1 in sweep
// t; each of the R = 2S-1 serial resources (stages, and one channel per stage pair for both
// directions) serves its items in (sweep, block) order, and an item starts when its
// microbatch has left block j-1 (which happened in sweep t-1) and the resource is idle:
//     fin_t[j] = max(fin_{t-1}[j-1], idle(resource of j)) + dur[j],
// where a resource's idle time is the latest finish of its two blocks j and 2R-j (finish
// times on one resource never decrease).  Within a sweep the forward block of a resource
// precedes its backward block.  T, the finish of the last backward block on stage 0, is the longest
// path through these items, which pp_makespan_path.h has in closed form: O(S) instructions for a plan
// whatever the microbatch counts, one lane per plan, all counts of a call together (up to four at a time).
//
// When asked to, each workgroup also reduces (T, candidate) to its minimum, and a one-workgroup
// kernel launched next reduces the minima to the winner record.
#include "pp_dp_flat.h"
#include "pp_makespan_path.h"

// One workgroup per microbatch count: the minimum (T, index) of its n_part partials, lowest
// index on ties, and the winner record.
__global__ __launch_bounds__(256) void k_pick(mk_args a) {
    __shared__ tc_pair sh[4];
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const tc_pair *part = a.part + (long long)q * a.n_part;
    tc_pair w = {PP_INF64, INT64_MAX};
    // four loads in flight per thread: the partials come straight from the kernel before, so
    // each round is a trip to memory
    const tc_pair none = {PP_INF64, INT64_MAX};
    for (long long i = tid; i < a.n_part; i += 1024) {
        tc_pair p0 = part[i];
        tc_pair p1 = i + 256 < a.n_part ? part[i + 256] : none;
        tc_pair p2 = i + 512 < a.n_part ? part[i + 512] : none;
        tc_pair p3 = i + 768 < a.n_part ? part[i + 768] : none;
        w = tc_min(tc_min(w, p0), tc_min(p1, tc_min(p2, p3)));
    }
    w = wave_tc_min(w);
    if (lane == 0) sh[tid >> 6] = w;
    __syncthreads();
    if (tid < 64) {
        w = tc_min(tc_min(sh[0], sh[1]), tc_min(sh[2], sh[3]));
        write_winner(a, q, w, lane);
    }
}

static int launch_pick(mk_args a, int nM, long long n_part, hipStream_t st) {
    a.n_part = n_part;
    hipLaunchKernelGGL(k_pick, dim3(nM), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}

// ---------------------------------------------------------------- plans in closed form, S <= 8

#define MK_FLAT_MAX_S 8

// LDS for plans built here: B and A of the channel-free program, PF and PB in pairs, the forward and backward
// channel time of every link; then per wave the words of mk_path_body, and per stage a lane's transfer times and the largest
// channel time so far.
__host__ __device__ static inline size_t mk_fuse_wave_bytes(int S) { return mk_path_wave_bytes(S) + (size_t)S * 64 * 12; }
__host__ __device__ static inline size_t mk_fuse_lds_bytes(int L, int D, int S, int waves) {
    return pp_flat_table_bytes(L, S) + mk_path_table_bytes(L) + (size_t)D * D * 8 + waves * mk_fuse_wave_bytes(S);
}

// When the plans are not in memory yet (a.fuse): if the tables say so (see mk_args), every lane builds its
// candidate's plan in closed form from tables staged in LDS - W[n][l] = max(largest channel time so far,
// channel-free cell), lowest split from the channel-free split table or by a search in the prefix sums - and takes
// the block durations from LDS as well, so that everything costs one trip to memory.  Returns false (nothing done)
// if this launch reads its plans from memory.
// What bounds it: that trip, and then the latency of loops over the stages (one wave per SIMD at 8! candidates).  Loops:
// straight-line code, which a wave runs once, waits for its instructions.
template <int NM>
__device__ __forceinline__ bool flat_body(const mk_args &a) {
    extern __shared__ __align__(16) int rows[];
    const int S = a.S, L = a.L, D = a.D, nP = L + 1, SP = S | 1, tid = threadIdx.x, lane = tid & 63, T = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = T >> 6;
    // requests first: header, the devices of this wave's candidates, the tables (contiguous in the workspace as B then
    // A), PF, PB, and the links' channel times
    const unsigned flat_w = a.hdr->flat[lane];
    const unsigned long long vmax = a.hdr->pmax[lane];
    long long g = (long long)blockIdx.x * waves + wave;
    int dev[MK_FLAT_MAX_S];
    auto fetch = [&](long long at) {
#pragma unroll
        for (int u = 0; u < MK_FLAT_MAX_S; ++u) {
            const long long t = at * 64 * S + u * 64 + lane;
            dev[u] = u < S && t < a.N * S ? a.orderings[t] : 0;
        }
    };
    fetch(g);
    const size_t tab = pp_flat_table_bytes(L, S);
    int *sB = rows, *sA = sB + (size_t)2 * S * nP;
    long long *PT = (long long *)((unsigned char *)rows + tab);
    int2 *links = (int2 *)(PT + 2 * nP);
    const int n16 = (int)(tab / 16);
    int4 first[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) first[u] = tid + u * T < n16 ? ((const int4 *)a.bfl)[tid + u * T] : make_int4(0, 0, 0, 0);
    // (what the first pass of the loops below stores)
    const long long pf0 = tid <= L ? a.PF[tid] : 0, pb0 = tid <= L ? a.PB[tid] : 0;
    const long long xf0 = tid < D * D && L > 1 ? a.XF[(size_t)tid * L] : 0, xb0 = tid < D * D && L > 1 ? a.XB[(size_t)tid * L] : 0;
    // (lane b holds the largest time of pack block b: all below the limit = their maximum is)
    const int limit = pp_time_limit(a.fuse_mmax, S);
    if (limit < 0 || __ballot(flat_w != 0) != ~0ull || __ballot(vmax > (unsigned long long)limit)) return false;
#pragma unroll
    for (int u = 0; u < 8; ++u)
        if (tid + u * T < n16) ((int4 *)sB)[tid + u * T] = first[u];
    for (int i = 8 * T + tid; i < n16; i += T) ((int4 *)sB)[i] = ((const int4 *)a.bfl)[i];  // (narrow workgroups)
    for (int i = tid; i <= L; i += T) {
        PT[2 * i] = i == tid ? pf0 : a.PF[i];
        PT[2 * i + 1] = i == tid ? pb0 : a.PB[i];
    }
    for (int i = tid; i < D * D; i += T)
        links[i] = make_int2((int)(i == tid ? xf0 : L > 1 ? a.XF[(size_t)i * L] : 0), (int)(i == tid ? xb0 : L > 1 ? a.XB[(size_t)i * L] : 0));
    int M[NM];
    bool briefly[NM];
    mk_counts<NM>(a, M);
    mk_briefly<PP_SCHED_PE>(M, S, briefly);
    tc_pair least[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) least[q] = {PP_INF64, INT64_MAX};
    const int steps = pp_flat_steps(L);
    int *mine = (int *)(links + D * D) + wave * (mk_fuse_wave_bytes(S) / 4), *row = mine + lane * SP;
    int2 *stash = (int2 *)(mine + mk_path_wave_bytes(S) / 4) + lane;
    int *most = (int *)(stash - lane + 64 * S) + lane;  // [n][64] largest channel time up to stage n
    __syncthreads();
    const int di = 64 / S, dn = 64 - di * S, i0 = lane / S, r0 = lane - i0 * S;
    for (; g * 64 < a.N; g += (long long)gridDim.x * waves) {
        const long long c = g * 64 + lane;
        const bool live = c < a.N;
        {
            int i = i0, n = r0;
#pragma unroll
            for (int u = 0; u < MK_FLAT_MAX_S; ++u) {
                if (u < S) mine[i * SP + n] = dev[u] >= 0 && dev[u] < D ? dev[u] : 0xffff;
                n += dn;
                i += di;
                if (n >= S) { n -= S; ++i; }
            }
        }
        fetch(g + (long long)gridDim.x * waves);  // (the next group's, on their way)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // a caller's row is checked here (the DP kernel has not looked at it)
        bool bad = false;
        int run = 0, before = 0;
        unsigned long long seen = 0;
#pragma unroll 1
        for (int n = 0; n < S; ++n) {
            int d = row[n];
            if (a.fuse_validate) {
                bad |= d >= D || (seen >> (d & 63) & 1);  // (D <= 32)
                seen |= 1ull << (d & 63);
                d = d < D ? d : 0;
            }
            if (n) {
                const int2 x = links[before * D + d];
                run = run > x.x + x.y ? run : x.x + x.y;
                stash[n * 64] = x;
                most[n * 64] = run;
            }
            before = d;
        }
        bad = bad && live;
        // the plan, from (S-1, L) downwards
        int e = L, C = 0;
#pragma unroll 1
        for (int n = S - 1; n >= 1; --n) {
            const int at = n * nP + e, bn = sB[2 * at], m = most[n * 64];
            int r = sA[at];
            if (n == S - 1) C = m > bn ? m : bn;
            row[n] = e;
            if (m > bn) {  // the channels bind: the longest last stage that fits in m
                const int t = sB[2 * e] - m;
                int pos = 0;
                for (int st = 1 << (steps - 1); st; st >>= 1) {
                    const int idx = pos + st - 1;
                    pos += sB[2 * (idx <= L ? idx : L)] < t ? st : 0;
                }
                r = pos < L ? pos : L;
                r = r > n ? r : n;
            }
            e = r;
        }
        row[0] = e;
        mk_path<int, NM> path;
        path.start();
        int f0 = (int)PT[0], b0 = (int)PT[1];
#pragma unroll 1
        for (int n = 0; n < S; ++n) {
            const int at = row[n];
            const int2 x = n ? stash[n * 64] : make_int2(0, 0);
            // (no time of the call leaves 32 bits: the low halves of the differences are the differences)
            const int f1 = (int)PT[2 * at], b1 = (int)PT[2 * at + 1], F = mk_less(f1, f0), B = mk_less(b1, b0);
            f0 = f1;
            b0 = b1;
            if (bad) row[n] = 0;
            mk_stage<PP_SCHED_PE>(path, n, S, F, B, x.x, x.y, M, briefly);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the plans go to memory (the winner's record is read from there, maybe by this workgroup)
        if (blockIdx.y == 0 || a.pick_here) {
            int i = i0, n = r0;
            for (int u = 0; u < S; ++u) {
                const long long t = g * 64 * S + u * 64 + lane;
                if (t < a.N * S) a.bounds_w[t] = mine[i * SP + n];
                n += dn;
                i += di;
                if (n >= S) { n -= S; ++i; }
            }
            if (live) a.C_w[c] = bad ? PP_INF64 : (long long)C;
        }
        __builtin_amdgcn_wave_barrier();
        if (bad) pp_raise(a.status, PP_FAULT_ORDERING);
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const int slot = (int)blockIdx.y * NM + q;
            if (slot >= a.nM || !live) continue;
            const long long t = bad ? PP_INF64 : (long long)path.longest(q);
            if (a.T_out) a.T_out[(long long)slot * a.N + c] = t;
            least[q] = tc_min(least[q], {t, c});
        }
    }
    mk_leave_least(a, least, (tc_pair *)rows);
    return true;
}

// pp_best_plan for 2 .. 8 stages: the plans from the tables without transfers where that is possible, else from memory.
template <int NM, bool FREE>
__global__ __launch_bounds__(64 * MK_PATH_WAVES) void k_makespan_flat(mk_args a) {
    if (!flat_body<NM>(a)) mk_path_body<PP_SCHED_PE, NM, true, FREE>(a);
}
template <bool FREE>
static void launch_flat(const mk_args &a, int counts, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (counts == 1) hipLaunchKernelGGL((k_makespan_flat<1, FREE>), grid, block, lds, st, a);
    else if (counts == 2) hipLaunchKernelGGL((k_makespan_flat<2, FREE>), grid, block, lds, st, a);
    else hipLaunchKernelGGL((k_makespan_flat<MK_COUNTS, FREE>), grid, block, lds, st, a);
}

static void plain_layout(mk_args &a, int S) {
    a.ord_stride = S; a.bnd_stride = S; a.bnd_off = 0; a.t_stride = 1; a.t_off = 0;
}

// The makespan kernel can build the plans itself (closed form, tables staged in LDS) for 2..8
// stages when its tables fit.
bool pp_makespan_can_fuse(int L, int D, int S) {
    return S >= 2 && S <= MK_FLAT_MAX_S && D <= 32 && mk_fuse_lds_bytes(L, D, S, 4) <= 64 * 1024;
}

// Everything of one call in one launch, and (with a.part) the winners.
static int launch_makespan(const mk_args &a, hipStream_t st) {
    long long n_part = 0;
    if (a.fuse) {
        const mk_path_launch l = mk_path_shape(a);
        const size_t need = mk_fuse_lds_bytes(a.L, a.D, a.S, l.waves), lds = need > l.lds ? need : l.lds;
        mk_args b = a;
        b.pick_here = l.pick;
        n_part = l.pick ? 0 : l.grid;
        const dim3 grid(l.grid, (a.nM + l.counts - 1) / l.counts), block(64 * l.waves);
        if (b.free_bits) launch_flat<true>(b, l.counts, grid, block, lds, st);
        else launch_flat<false>(b, l.counts, grid, block, lds, st);
        if (hipGetLastError() != hipSuccess) return PP_ERR_HIP;
    } else {
        const int rc = pp_launch_makespan_split(a, st, &n_part);
        if (rc) return rc;
    }
    return a.part && n_part ? launch_pick(a, a.nM, n_part, st) : PP_OK;
}

int pp_launch_makespan(int L, int D, int S, int64_t N, int nM, const int *Ms, const int64_t *PF,
                       const int64_t *PB, const int64_t *XF, const int64_t *XB,
                       const int32_t *orderings, const int32_t *bounds, int64_t *T_out,
                       int32_t *status, const int64_t *C, void *part,
                       pp_result *out, const pp_ws_header *hdr, const pp_fuse_info *fuse,
                       const int32_t *rlist, const pp_free_plans *done, hipStream_t st) {
    if (rlist && (!hdr || !part)) return PP_ERR_INVALID_ARG;
    mk_args a = {};
    a.rlist = rlist;
    a.L = L; a.D = D; a.S = S; a.N = N;
    a.nM = nM;
    for (int q = 0; q < PP_MAX_M_LIST; ++q) a.Ms[q] = q < nM ? Ms[q] : 1;
    a.PF = (const long long *)PF; a.PB = (const long long *)PB;
    a.XF = (const long long *)XF; a.XB = (const long long *)XB;
    a.orderings = orderings; a.bounds = bounds;
    plain_layout(a, S);
    a.T_out = (long long *)T_out; a.status = status;
    a.part = (tc_pair *)part; a.C = (const long long *)C; a.out = out;
    a.hdr = hdr;
    if (done && hdr && part) {
        a.free_bits = done->bits;
        a.free_least = done->least;
        a.free_plan = done->plan;
    }
    if (fuse && hdr && !rlist && pp_makespan_can_fuse(L, D, S)) {
        a.fuse = 1;
        a.fuse_mmax = fuse->mmax;
        a.fuse_validate = fuse->validate;
        a.bfl = (const long long *)fuse->bfl;
        a.C_w = (long long *)fuse->C;
        a.bounds_w = fuse->bounds;
    }
    return launch_makespan(a, st);
}

// ---------------------------------------------------------------- stage-count search

int pp_launch_makespan_stages(int L, int D, int S, int64_t N, int nM, const int *Ms,
                              const int64_t *PF, const int64_t *PB, const int64_t *XF,
                              const int64_t *XB, const int32_t *orderings, const int32_t *bounds,
                              const int64_t *C, int64_t *T_st, int32_t *status, void *part,
                              pp_result *out, const pp_ws_header *hdr,
                              const int32_t *rlist, hipStream_t st) {
    if (rlist && !hdr) return PP_ERR_INVALID_ARG;
    mk_args a = {};
    a.rlist = rlist;
    a.L = L; a.D = D; a.S = S; a.N = N; a.nM = nM;
    for (int q = 0; q < PP_MAX_M_LIST; ++q) a.Ms[q] = q < nM ? Ms[q] : 1;
    a.PF = (const long long *)PF; a.PB = (const long long *)PB;
    a.XF = (const long long *)XF; a.XB = (const long long *)XB;
    a.orderings = orderings; a.bounds = bounds;
    a.T_out = (long long *)T_st; a.status = status;
    a.part = (tc_pair *)part; a.C = (const long long *)C; a.out = out;
    a.ord_stride = S; a.bnd_stride = (long long)S * (S + 1) / 2; a.t_stride = S;
    a.search = S;
    a.hdr = hdr;
    return launch_makespan(a, st);
}

// ---------------------------------------------------------------- replicated stages: launch

int pp_launch_rep_makespan(int L, int D, int64_t N, int M, const int64_t *PF, const int64_t *PB,
                           const int64_t *PA, const int64_t *actf, const int64_t *actb,
                           const int64_t *bw, const int32_t *orderings, const int32_t *bounds,
                           const int32_t *reps, const int64_t *W, int64_t *T_out, int32_t *status,
                           void *part, pp_rep_result *out, hipStream_t st) {
    if (D > 16) return PP_ERR_INVALID_ARG;
    mk_args a = {};
    a.L = L; a.D = D; a.N = N; a.nM = 1;
    for (int q = 0; q < PP_MAX_M_LIST; ++q) a.Ms[q] = M;
    a.PF = (const long long *)PF; a.PB = (const long long *)PB;
    a.XF = a.XB = NULL;
    a.PA = (const long long *)PA; a.actf = (const long long *)actf; a.actb = (const long long *)actb;
    a.bw = (const long long *)bw; a.W = (const long long *)W;
    a.orderings = orderings; a.bounds = bounds; a.reps = reps;
    a.T_out = (long long *)T_out; a.status = status;
    a.ord_stride = D; a.bnd_stride = (long long)D * (D + 1) / 2; a.t_stride = D;
    a.S = D; a.search = D;
    a.part = (tc_pair *)part; a.C = (const long long *)W; a.rout = out;
    long long n_part = 0;
    const int rc = mk_launch_replicated(a, st, &n_part);
    return rc || !n_part ? rc : launch_pick(a, 1, n_part, st);
}

// ---------------------------------------------------------------- schedule variants

// Checks candidate c's ordering and bounds and gathers its block durations through `put`
// (called as put(block j (1-based), duration)).  Returns fault bits; on a fault or for a
// dead lane all durations are 0.  `worst` gets the largest per-resource time f + b.
template <typename Put>
__device__ __forceinline__ int gather_durations(const mk_args &a, long long c, bool live, long long &worst, Put put) {
    const int S = a.S, L = a.L, D = a.D, R = 2 * S - 1;
    int fault = 0;
    if (live) {
        if (a.orderings) {
            for (int n = 0; n < S; ++n) {
                int d = a.orderings[c * a.ord_stride + n];
                bool bad = d < 0 || d >= D;
                for (int q = 0; q < n; ++q) bad |= (a.orderings[c * a.ord_stride + q] == d);
                if (bad) fault |= PP_FAULT_ORDERING;
            }
        }
        // (a bad ordering is reported alone: its plan is not looked at)
        int prev = 0, fb = 0;
        for (int n = 0; n < S; ++n) {
            int e = a.bounds[c * a.bnd_stride + a.bnd_off + n];
            if (e <= prev || e > L) fb = PP_FAULT_BOUNDS;
            prev = e;
        }
        if (prev != L) fb = PP_FAULT_BOUNDS;
        fault = fault ? fault : fb;
    }
    worst = 0;
    unsigned long long rem = (unsigned long long)(live ? c : 0);
    unsigned used = 0;
    int e_prev = 0, o_prev = 0;
    for (int n = 0; n < S; ++n) {
        long long F = 0, Bk = 0, cf = 0, cb = 0;
        if (live && !fault) {
            int o_n = a.orderings ? a.orderings[c * a.ord_stride + n] : pp_unrank_next(D, n, rem, used);
            int e = a.bounds[c * a.bnd_stride + a.bnd_off + n];
            F = a.PF[e] - a.PF[e_prev];
            Bk = a.PB[e] - a.PB[e_prev];
            if (n) {
                size_t at = ((size_t)o_prev * D + o_n) * L + (size_t)(e_prev - 1);
                cf = a.XF[at];
                cb = a.XB[at];
            }
            e_prev = e;
            o_prev = o_n;
        }
        long long w = F + Bk > cf + cb ? F + Bk : cf + cb;
        worst = w > worst ? w : worst;
        const int r = 2 * n + 1;  // stage n is resource 2n+1, channel n is resource 2n
        if (n == S - 1) {
            put(R, F + Bk);  // merged forward+backward block of the last stage
        } else {
            put(r, F);
            put(2 * R - r, Bk);
        }
        if (n) {
            put(r - 1, cf);
            put(2 * R - (r - 1), cb);
        }
    }
    return fault;
}

// PP_SCHED_FIFO in general, any S, 64 bits, one lane per candidate, the lane's state in its own LDS column (rows
// [row][lane]): Alg. 1 with channels that serve by readiness instead of by list (only computation blocks enter the
// lists U_s in the listing), as an event simulation.  It does the candidates that k_makespan_fifo, launched before it,
// has marked: long times, zero durations and more than 32 stages (by_block == 0: all candidates).
__global__ __launch_bounds__(64) void k_makespan_events(mk_args a) {
    extern __shared__ long long sm[];
    const int lane = threadIdx.x, W = blockDim.x;
    const long long c = (long long)blockIdx.x * W + lane;
    const bool live = c < a.N && (!a.by_block || a.T_out[c] == MK_NOT_TAKEN);
    if (!__ballot(live)) return;
    const int S = a.S, M = a.Ms[0];
    const int R = 2 * S - 1, J = 2 * R - 1;
    long long *dur = sm + lane;                    // rows 0..J-1: duration of block j = row + 1
    long long worst;
    const int fault0 = gather_durations(a, c, live, worst, [&](int j, long long d) { dur[(size_t)(j - 1) * W] = d; });
    const int fault = (live && !fault0) ? overflow_fault(worst, M, S) : fault0;
    // One committed item per iteration (the same in every lane): every
    // block handles the microbatches in index order, nxt[j] is block j's next one.  A
    // stage's next item is the earlier of its two blocks' heads in list order (sweep
    // m + j - 1, then block); a channel takes, of its heads whose microbatch has left the
    // preceding block, the one that left it first (equal: earlier in list order).  The item
    // with the earliest start over all resources is committed (equal: lowest resource).
    // A microbatch is in exactly one place, so one "left its last block at" time per
    // microbatch in flight is enough; the first stage's list keeps at most J in flight,
    // so they live in a ring of Q >= J slots (Q a power of two).
    int Q = 1;
    while (Q < J) Q <<= 1;
    long long *idle = sm + (size_t)J * W + lane;        // rows J..J+R-1: resource r at r-1
    long long *ring = idle + (size_t)R * W;             // Q rows
    long long *nxt = ring + (size_t)Q * W;              // J rows: block j at j-1
    for (int r = 0; r < R; ++r) idle[(size_t)r * W] = 0;
    for (int q = 0; q < Q; ++q) ring[(size_t)q * W] = 0;
    for (int j = 0; j < J; ++j) nxt[(size_t)j * W] = 1;
    long long T = 0;
    for (long long left = (long long)J * M; left > 0; --left) {
        int best_r = 0, best_j = 0;
        long long best_start = 0;
        for (int r = 1; r <= R; ++r) {
            const int ja = r, jb = 2 * R - r;
            const int ma = (int)nxt[(size_t)(ja - 1) * W], mb = (int)nxt[(size_t)(jb - 1) * W];
            // head (m, j) of a block is there once block j-1 has moved past m
            const bool at_a = ma <= M && (ja == 1 || (int)nxt[(size_t)(ja - 2) * W] > ma);
            const bool at_b = jb != ja && mb <= M && (int)nxt[(size_t)(jb - 2) * W] > mb;
            const long long ra = ja == 1 ? 0 : ring[(size_t)(ma & (Q - 1)) * W];
            const long long rb = ring[(size_t)(mb & (Q - 1)) * W];
            int j = 0;
            if (r & 1) {
                const bool has_a = ma <= M, has_b = jb != ja && mb <= M;
                if (has_a && (!has_b || ma + ja <= mb + jb)) j = at_a ? ja : 0;
                else if (has_b) j = at_b ? jb : 0;
            } else {
                const bool a_first = ra < rb || (ra == rb && ma + ja <= mb + jb);
                if (at_a && (!at_b || a_first)) j = ja;
                else if (at_b) j = jb;
            }
            const long long ready = j == ja ? ra : rb;
            const long long busy = idle[(size_t)(r - 1) * W];
            const long long start = ready > busy ? ready : busy;
            if (j && (!best_r || start < best_start)) { best_r = r; best_j = j; best_start = start; }
        }
        // (there always is one: block 1 or the successor of a finished item)
        if (best_r) {
            const long long f = best_start + dur[(size_t)(best_j - 1) * W];
            const int m = (int)nxt[(size_t)(best_j - 1) * W];
            ring[(size_t)(m & (Q - 1)) * W] = f;
            idle[(size_t)(best_r - 1) * W] = f;
            nxt[(size_t)(best_j - 1) * W] = m + 1;
            if (best_j == J) T = f > T ? f : T;
        }
    }
    if (live) {
        if (fault) pp_raise(a.status, fault);
        a.T_out[c] = fault ? PP_INF64 : T;
    }
}

int pp_launch_makespan_variant(int variant, int L, int D, int S, int64_t N, int M, const int64_t *PF,
                               const int64_t *PB, const int64_t *XF, const int64_t *XB,
                               const int32_t *orderings, const int32_t *bounds, int64_t *T_out,
                               int32_t *status, hipStream_t st) {
    mk_args a = {};
    a.L = L; a.D = D; a.S = S; a.N = N; a.nM = 1;
    for (int q = 0; q < PP_MAX_M_LIST; ++q) a.Ms[q] = M;
    a.PF = (const long long *)PF; a.PB = (const long long *)PB;
    a.XF = (const long long *)XF; a.XB = (const long long *)XB;
    a.orderings = orderings; a.bounds = bounds;
    plain_layout(a, S);
    a.variant = variant;
    a.T_out = (long long *)T_out; a.status = status;
    if (variant != PP_SCHED_FIFO) return pp_launch_makespan_split(a, st);
    // The faster kernel pays where a schedule is long enough for a second launch, and where there is a
    // pipeline.  10 plans, the general kernel alone / both (with the three other schedules of that time in one sum), us:
    // S = 1 40 / 49 (M = 4 and 32) and 10^6 plans 1018 / 1457 (M = 256); S = 2, M = 4 40 / 51; S = 3, M = 4 80 / 51;
    // S = 2, M = 32 215 / 81.
    // (Lists with plans the readiness order leaves to the general kernel - items of zero length - S = 2, M = 32,
    // 20 000 plans 223 / 197; S = 3, M = 4 84 / 92.)
    a.by_block = S <= 32 && S > 1 && (long long)(4 * S - 3) * M > 24;
    if (a.by_block) {
        const int rc = pp_launch_makespan_fifo(a, st);
        if (rc) return rc;
    }
    // durations, resource idle times, a power-of-two ring of J or more, next microbatches
    const int J = 4 * S - 3, R = 2 * S - 1;
    int Q = 1, W = 64;
    while (Q < J) Q <<= 1;
    const size_t rows = (size_t)J + R + Q + J;
    while (rows * W * 8 > 64 * 1024) W >>= 1;
    hipLaunchKernelGGL(k_makespan_events, dim3((unsigned)((N + W - 1) / W)), dim3(W), rows * W * 8, st, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
