// The schedules of plans in memory under every order but the readiness one: T by the closed form of
// pp_makespan_path.h, one lane per plan.
//
// What bounds it: the scattered reads of the links' transfer times, two per stage, then instruction issue (about 12 and
// 14 per microbatch count for each of the 2 S - 1 resources).  A sweep over all blocks per microbatch, which this
// replaces, issued 4 to 5 instructions per (resource, sweep).  Whole calls, before and after: 131 071 plans of 32
// stages, M = 64 and 128 600 -> 67 us; the search over 2^20 orderings with 32 stages, M = 128 2.77 -> 0.73 ms, over
// 200 003 with 11 stages, M = 10 and 33 162 -> 79 us.
#include "pp_makespan_path.h"

template <int MODE, int NM>
__global__ __launch_bounds__(64 * MK_PATH_WAVES) void k_makespan_split(mk_args a) {
    mk_path_body<MODE, NM, false>(a);
}
// (FREE in a kernel of its own: with four counts the other has 121 registers, four waves per SIMD, and takes 28 us for
// the plans of every stage count of 8! orderings, 41 with 131)
template <int NM, bool FREE>
__global__ __launch_bounds__(64 * MK_PATH_WAVES) void k_makespan_plans(mk_args a) {
    mk_path_body<PP_SCHED_PE, NM, true, FREE>(a);
}
template <bool FREE>
static void launch_plans(const mk_args &a, const mk_path_launch &l, dim3 grid, dim3 block, hipStream_t st) {
    if (l.counts == 1) hipLaunchKernelGGL((k_makespan_plans<1, FREE>), grid, block, l.lds, st, a);
    else if (l.counts == 2) hipLaunchKernelGGL((k_makespan_plans<2, FREE>), grid, block, l.lds, st, a);
    else hipLaunchKernelGGL((k_makespan_plans<MK_COUNTS, FREE>), grid, block, l.lds, st, a);
}

int pp_launch_makespan_split(const mk_args &a, hipStream_t st, long long *n_part) {
    const mk_path_launch l = mk_path_shape(a);
    mk_args b = a;
    b.pick_here = l.pick;
    if (n_part) *n_part = l.pick ? 0 : l.grid;
    const dim3 grid(l.grid, (a.nM + l.counts - 1) / l.counts), block(64 * l.waves);
    if (a.hdr) {
        // (inside the planner)
        if (b.free_bits) launch_plans<true>(b, l, grid, block, st);
        else launch_plans<false>(b, l, grid, block, st);
        return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
    }
    switch (a.variant) {
        case PP_SCHED_PE:
            if (l.counts == 1) hipLaunchKernelGGL((k_makespan_split<PP_SCHED_PE, 1>), grid, block, l.lds, st, b);
            else if (l.counts == 2) hipLaunchKernelGGL((k_makespan_split<PP_SCHED_PE, 2>), grid, block, l.lds, st, b);
            else hipLaunchKernelGGL((k_makespan_split<PP_SCHED_PE, MK_COUNTS>), grid, block, l.lds, st, b);
            break;
        // (the comparison schedules take one count)
        case PP_SCHED_DUPLEX: hipLaunchKernelGGL((k_makespan_split<PP_SCHED_DUPLEX, 1>), grid, block, l.lds, st, b); break;
        case PP_SCHED_GPIPE: hipLaunchKernelGGL((k_makespan_split<PP_SCHED_GPIPE, 1>), grid, block, l.lds, st, b); break;
        case PP_SCHED_ADDITIVE: hipLaunchKernelGGL((k_makespan_split<PP_SCHED_ADDITIVE, 1>), grid, block, l.lds, st, b); break;
        default: return PP_ERR_INVALID_ARG;
    }
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
