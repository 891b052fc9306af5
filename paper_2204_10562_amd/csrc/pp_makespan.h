// What the makespan kernels share: arguments, the arg-min's pairs, the way results go out.
#pragma once

#include "pp_common.h"

struct tc_pair { long long T, c; };

struct mk_args {
    int L, D, S, nM;
    int Ms[PP_MAX_M_LIST];  // microbatch counts; the plans are evaluated once per entry
    long long N;
    const long long *PF, *PB, *XF, *XB;
    const int *orderings;  // NULL = all D! orderings, candidate index = lexicographic rank
    const int *bounds;
    long long *T_out;      // [nM][N]; may be NULL when only the winners are wanted
    // Where candidate c's data lie: devices at orderings[c*ord_stride + n], bounds at
    // bounds[c*bnd_stride + bnd_off + n], T of microbatch count q at
    // T_out[(q*N + c)*t_stride + t_off].  (ord_stride, bnd_stride, bnd_off, t_stride, t_off)
    // = (S, S, 0, 1, 0) for plain lists; the stage-count search evaluates the plans with S = xi
    // stages out of rows that hold search = S_max devices and all S_max plans.
    int ord_stride, bnd_off, t_off;
    long long bnd_stride, t_stride;
    // search > 0: the plans of every stage count xi = 1 .. search of N candidates; the arg-min runs over the
    // pairs, entry c*search + xi-1, and the record of the winner is decoded accordingly
    int search;
    int variant;  // PP_SCHED_*
    // k_makespan_events: nonzero = only the candidates that k_makespan_fifo has marked (MK_NOT_TAKEN in T_out)
    int by_block;
    int lanes_per;  // lanes per candidate of k_makespan_fifo (1 .. 32)
    int groups;     // candidates per workgroup of k_makespan_fifo
    long long first;  // k_makespan_fifo: the launch's first candidate
    // workspace header, where the plans are the planner's own (C is there then); NULL: the caller's plans
    const pp_ws_header *hdr;
    // k_makespan_flat inside pp_best_plan: nonzero = when no link's channel time depends on the
    // cut position and every finish time of the launch fits 32 bits (both read from hdr), the
    // partition DP kernel has left the plans to this kernel, which builds them in closed form
    // from the channel-free tables bfl (pp_dp_flat.h) and writes C_w [N] and bounds_w [N][S].
    // fuse_mmax: the largest microbatch count of the call (the DP kernel tests the same bound).
    int fuse, fuse_mmax, fuse_validate;
    const long long *bfl;
    long long *C_w;
    int *bounds_w;
    int32_t *status;
    // replicated stages (k_rep_makespan and the record of its arg-min; NULL otherwise): replica
    // counts laid out like bounds, prefix sums of the parameter sizes, activation sizes, the
    // bandwidth matrix, and W per (candidate, stage count) (PP_INF64 = no such plan)
    const int *reps;
    const long long *PA, *actf, *actb, *bw, *W;
    // inside pp_best_plan: non-NULL = if the workspace header says that candidates share their
    // partition DP (pp_share.hip), this is the list of the candidates that stand for all others;
    // only they are scheduled
    const int *rlist;
    // plans that k_band_free has scheduled (pp_free_plans), or NULL
    const unsigned long long *free_bits;
    const long long *free_least;
    const int *free_plan;
    pp_rep_result *rout;   // [nM] winner records with replica counts (instead of out)
    // arg-min (all NULL when not wanted)
    tc_pair *part;         // [nM][workgroups]: every workgroup's minimum, reduced by k_pick
    long long n_part;      // k_pick: partials per microbatch count
    int pick_here;         // the launch is one workgroup, which writes the records itself
    const long long *C;
    pp_result *out;        // [nM]
};

__device__ __forceinline__ tc_pair tc_min(tc_pair a, tc_pair b) {
    return (b.T < a.T || (b.T == a.T && b.c < a.c)) ? b : a;
}

// Over the wave's lanes: four steps within each row of 16 (quad_perm, half_mirror, mirror), then the four rows.
template <int CTRL>
__device__ __forceinline__ tc_pair tc_step(tc_pair v) {
    auto from = [](long long x) {
        const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, 0xf, 0xf, true);
        return (long long)((unsigned long long)(unsigned)hi << 32 | (unsigned)lo);
    };
    return tc_min(v, {from(v.T), from(v.c)});
}
__device__ __forceinline__ tc_pair wave_tc_min(tc_pair v) {
    v = tc_step<0x140>(tc_step<0x141>(tc_step<0x4E>(tc_step<0xB1>(v))));
    auto row = [&](int i) {
        auto at = [&](long long x) {
            const int lo = __builtin_amdgcn_readlane((int)x, i), hi = __builtin_amdgcn_readlane((int)(x >> 32), i);
            return (long long)((unsigned long long)(unsigned)hi << 32 | (unsigned)lo);
        };
        return tc_pair{at(v.T), at(v.c)};
    };
    return tc_min(tc_min(row(0), row(16)), tc_min(row(32), row(48)));
}

// The schedule is no longer than (M + 4S - 4) * C (Lemma 1): fault if that bound reaches 2^62.
__device__ __forceinline__ int overflow_fault(long long worst, int M, int S) {
    return worst > (PP_CAP62 - 1) / ((long long)M + 4 * S - 4) ? PP_FAULT_OVERFLOW : 0;
}

// T of a candidate that k_makespan_fifo has left to k_makespan_events (no schedule ends before 0).
#define MK_NOT_TAKEN (-1ll)
// Whether k_band_free has scheduled candidate c.  (It has not looked at any where candidates share their DP.)
__device__ __forceinline__ bool mk_has_free(const mk_args &a) { return a.free_bits && a.hdr->free_valid; }
__device__ __forceinline__ bool mk_is_free(const mk_args &a, long long c) {
    return mk_has_free(a) && (a.free_bits[c >> 6] >> (c & 63) & 1);
}

// The winner record of microbatch count q from the minimum w over all entries.
__device__ __forceinline__ void write_winner(const mk_args &a, int q, tc_pair w, int lane) {
    const int S = a.S;
    const bool none = w.T == PP_INF64;
    // the winner: candidate c with xi stages, its C at C[at_c], its bounds from bounds[at_b]
    long long c = w.c, at_c = w.c, at_b = w.c * a.bnd_stride + a.bnd_off;
    int xi = S;
    if (a.search && !none) {
        c = w.c / a.search;
        xi = (int)(w.c - c * a.search) + 1;
        at_b = c * ((long long)a.search * (a.search + 1) / 2) + xi * (xi - 1) / 2;
    }
    if (a.rout) {
        // plan with replicated stages: xi bounds and replica counts, all D devices by rank
        pp_rep_result *out = a.rout + q;
        if (lane == 0) {
            out->best_index = none ? -1 : c;
            out->T = w.T;
            out->W = none ? PP_INF64 : a.C[at_c];
            out->S = none ? 0 : xi;
        }
        const bool in = lane < xi && !none;
        out->bounds[lane] = in ? a.bounds[at_b + lane] : 0;
        out->reps[lane] = in ? a.reps[at_b + lane] : 0;
        out->order[lane] = (lane < a.D && !none) ? a.orderings[c * a.ord_stride + lane] : 0;
        return;
    }
    pp_result *out = a.out + q;
    if (lane == 0) {
        out->best_index = none ? -1 : c;
        out->T = w.T;
        out->C = none ? PP_INF64 : a.C[at_c];
        out->S = xi;
    }
    // lane n writes bound n and device n (lanes xi.. write zeros)
    int b = 0, o = 0;
    if (lane < xi && !none) {
        b = mk_is_free(a, c) ? a.free_plan[lane] : a.bounds[at_b + lane];
        if (a.orderings) {
            o = a.orderings[c * a.ord_stride + lane];
        } else {
            unsigned long long rem = (unsigned long long)c;
            unsigned used = 0;
            for (int n = 0; n <= lane; ++n) o = pp_unrank_next(a.D, n, rem, used);
        }
    }
    out->bounds[lane] = b;
    out->order[lane] = o;
}

// Fault bits of a candidate whose devices and bounds lie in LDS (o: filled in for the list of all D!
// orderings).  A bad ordering is reported alone: its plan is not looked at.
__device__ __forceinline__ int mk_check_rows(const mk_args &a, long long c, int *o, const int *e) {
    const int S = a.S, L = a.L, D = a.D;
    if (a.orderings) {
        unsigned long long seen = 0;
        bool bad = false;
        for (int n = 0; n < S; ++n) {
            const int d = o[n];
            bad |= d < 0 || d >= D;
            if (D <= 64) {
                bad |= (seen >> (d & 63)) & 1;
                seen |= 1ull << (d & 63);
            } else {
                for (int q = 0; q < n; ++q) bad |= o[q] == d;
            }
        }
        if (bad) return PP_FAULT_ORDERING;
    } else {
        unsigned long long rem = (unsigned long long)c;
        unsigned used = 0;
        for (int n = 0; n < S; ++n) o[n] = pp_unrank_next(D, n, rem, used);
    }
    int prev = 0, fault = 0;
    for (int n = 0; n < S; ++n) {
        if (e[n] <= prev || e[n] > L) fault = PP_FAULT_BOUNDS;
        prev = e[n];
    }
    return prev != L ? PP_FAULT_BOUNDS : fault;
}

// The longest path's closed form (pp_makespan_path.h) over the plans in memory, any a.variant but PP_SCHED_FIFO
// (pp_makespan_split.hip).  With a.part it leaves partials for k_pick, *n_part of them per count, or picks itself
// (*n_part = 0).
int pp_launch_makespan_split(const mk_args &a, hipStream_t st, long long *n_part = NULL);
// PP_SCHED_FIFO for at most 32 stages (pp_makespan_fifo.hip); marks the candidates it leaves alone.
int pp_launch_makespan_fifo(const mk_args &a, hipStream_t st);

// The schedules of all plans with replicated stages: 1..a.D stages, a.N candidates
// (pp_makespan_rep.hip), and partials for k_pick as pp_launch_makespan_split leaves them.
int mk_launch_replicated(const mk_args &a, hipStream_t st, long long *n_part);

