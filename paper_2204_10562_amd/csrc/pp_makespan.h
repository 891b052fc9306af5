// What the makespan kernels share: arguments, the arg-min's pairs, the way results go out.
#pragma once

#include "pp_common.h"

struct tc_pair { long long T, c; };

struct mk_args {
    int L, D, S, nM;
    int Ms[PP_MAX_M_LIST];  // microbatch counts; the plans are evaluated once per entry
    // k_makespan_regs: wave slot i (blockIdx.y * waves + wave) serves count Ms[order[i]]
    unsigned char order[PP_MAX_M_LIST];
    // k_makespan_regs8: a workgroup holds `groups` groups of waves, each group one wave per
    // microbatch count for its own 64 candidates; wave w of group g takes slot
    // (slot_perm >> 2 (4 g + w)) & 3 of its four
    int groups;
    unsigned slot_perm;
    // k_makespan_regs8: nonzero = blockIdx.z + 1 is the number of stages xi, the plan with xi
    // stages is read from the triangular bounds array and T goes to column xi-1 (S, bnd_off and
    // t_off are then ignored)
    int all_xi;
    // With all_xi and the library's own list of all D! orderings in lexicographic order:
    // share[xi] = (D - xi)! consecutive candidates share their first xi devices and with them
    // the plan of xi stages, so it is scheduled once per such block (share[xi] = 1: no sharing)
    long long share[9];
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
    // search > 0 (arg-min only): the N entries are (candidate, stage count) pairs, entry
    // i = c*search + xi-1; the record of the winner is decoded accordingly
    int search;
    int variant;  // k_makespan_variant only: PP_SCHED_*
    // k_makespan_split / k_makespan_lds launched together without a header (more than 16 stages, no
    // workspace): nonzero = every block of 64 candidates decides for itself which of the two
    // kernels schedules it; k_makespan_split leaves MK_NOT_TAKEN in T_out of those it does not take
    int by_block;
    int lanes_per;  // lanes per candidate of k_makespan_split (1, 2, 4 or 8) and k_makespan_fifo (1 .. 64)
    long long first;  // k_makespan_fifo: the launch's first candidate
    // workspace header with the largest time of the tables (NULL if there is none): lets every
    // wave of a launch take the same decision between 32-bit and 64-bit finish times
    const pp_ws_header *hdr;
    // k_makespan_regs8 inside pp_best_plan: nonzero = when no link's channel time depends on the
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
    // k_makespan_regs<S> inside pp_best_plan: non-NULL = if the workspace header says that
    // candidates share their partition DP (pp_share.hip), this is the list of the candidates
    // that stand for all others; only they are scheduled (entry i by lane i of the launch), and
    // the slots of the partials no wave writes hold "none" already
    const int *rlist;
    pp_rep_result *rout;   // [nM] winner records with replica counts (instead of out)
    // arg-min (all NULL when not wanted)
    tc_pair *part;         // [nM][waves]: every wave's minimum, reduced by k_pick
    long long n_part;      // k_pick: partials per microbatch count
    const long long *C;
    pp_result *out;        // [nM]
};

__device__ __forceinline__ tc_pair tc_min(tc_pair a, tc_pair b) {
    return (b.T < a.T || (b.T == a.T && b.c < a.c)) ? b : a;
}

__device__ __forceinline__ tc_pair wave_tc_min(tc_pair v) {
    for (int off = 32; off; off >>= 1) {
        tc_pair o;
        o.T = __shfl_xor(v.T, off);
        o.c = __shfl_xor(v.c, off);
        v = tc_min(v, o);
    }
    return v;
}

// The schedule is no longer than (M + 4S - 4) * C (Lemma 1): fault if that bound reaches 2^62.
__device__ __forceinline__ int overflow_fault(long long worst, int M, int S) {
    return worst > (PP_CAP62 - 1) / ((long long)M + 4 * S - 4) ? PP_FAULT_OVERFLOW : 0;
}

// Writes T of microbatch count q, raises faults, and returns the wave's minimum.
__device__ __forceinline__ tc_pair emit_T(const mk_args &a, int q, long long c, bool live, int fault, long long T, int t_off) {
    if (live) {
        if (fault) { T = PP_INF64; pp_raise(a.status, fault); }
        if (a.T_out) a.T_out[((long long)q * a.N + c) * a.t_stride + t_off] = T;
    }
    tc_pair v = {live ? T : PP_INF64, live ? c : INT64_MAX};
    return a.part ? wave_tc_min(v) : v;
}

// The same, and (if wanted) leaves the wave's minimum in its slot of the partials; k_pick, launched next on the
// same stream, reduces the partials.
// (Plain stores and a kernel boundary: earlier versions let the last wave to arrive do the
// final reduction, but the returned atomics and arrival counters that needs cost more than
// the schedule itself once a launch has thousands of waves.)
__device__ __forceinline__ void emit(const mk_args &a, int q, long long c, bool live, int fault,
                                     long long T, long long wave_id, long long n_waves, int t_off) {
    const tc_pair v = emit_T(a, q, c, live, fault, T, t_off);
    if (!a.part) return;
    if ((threadIdx.x & 63) == 0 && wave_id < n_waves) a.part[(long long)q * n_waves + wave_id] = v;
}

// T of a candidate that k_makespan_split has left to k_makespan_lds (no schedule ends before 0).
#define MK_NOT_TAKEN (-1ll)
// Largest finish time k_makespan_split works with.
#define MK_SPLIT_CAP 0x3fffffff
// True if every finish time of a pipeline of S stages whose largest per-resource time is `worst`
// stays below MK_SPLIT_CAP for M microbatches (Lemma 1, with the sweeps of the padded pipeline), and
// the number of sweeps fits an int also where all times are zero.
__device__ __forceinline__ bool mk_split_fits(long long worst, long long M, int S) {
    return M + 4 * S + 64 <= MK_SPLIT_CAP && worst <= MK_SPLIT_CAP / (M + 4 * S + 64);
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

// Resources over lanes (pp_makespan_split.hip): times below MK_SPLIT_CAP, a.variant any but
// PP_SCHED_FIFO.  With a.by_block it marks the candidates it leaves alone.
int pp_launch_makespan_split(const mk_args &a, hipStream_t st);
// PP_SCHED_FIFO for at most 32 stages (pp_makespan_fifo.hip); marks the candidates it leaves alone.
int pp_launch_makespan_fifo(const mk_args &a, hipStream_t st);

// The schedules of all plans with replicated stages: 1..a.D stages, a.N candidates
// (pp_makespan_rep.hip).
int mk_launch_replicated(const mk_args &a, hipStream_t st);
