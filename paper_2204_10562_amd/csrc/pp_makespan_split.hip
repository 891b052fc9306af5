// Makespan for more than 16 stages, and the comparison schedules for any number but PP_SCHED_FIFO, with
// times below 2^30: the resources of a candidate spread over
// 1, 2, 4 or 8 neighbouring lanes, every finish time and duration in a register.
//
// The recurrence is that of pp_makespan.hip: in sweep t resource r = 1..R (R = 2S - 1; odd: stages,
// even: channels) serves its forward item and then its backward item,
//     f_t[r] = max(idle(r), f_{t-1}[r-1]) + df[r],   b_t[r] = max(idle(r), b_{t-1}[r+1]) + db[r],
// idle(r) being the later of the two's latest finishes; the merged block R is f[R] alone and is what
// resource R - 1 takes as b[R].  A lane holds RL consecutive resources, so a sweep is straight-line
// code over registers plus two lane shifts (f of the lane before, b of the lane after).  With G lanes
// per candidate the first G RL - R places are empty: their forward side passes the source through
// (df = 0, which delays every microbatch by as many sweeps) and their backward side stays negative
// (db = -2^30), so that the source enters at place 0 and block R sits at the last place whatever S.
//
// A place without an item in a sweep must leave its resource alone.  Values below zero mark such
// places, and the kinds of sweeps differ in where they can be:
//   filling (t <= M, not every resource has a backward item yet): forward places that are not
//     reached yet run through negative numbers by themselves (they start at -2^30 and the sums of
//     durations stay below 2^30); a backward place whose input is negative hands its sign on (a time
//     with that sign is a number from -2^31 up).  The resource is idle from max(f, b): 5 instructions
//     per resource.
//   full: 4 instructions per resource, f = max(b, f') + df, b = max(f, b') + db.
//   draining (t > M, the source gives -2^30): a forward place whose input is negative hands its sign
//     on; b, which is served in every sweep by now, says when the resource is idle: 5 instructions.
//     Backward places that are through run on into numbers nobody reads.
//   both (M smaller than the pipeline is deep): the idle times are kept apart: 8 instructions.
//
// What bounds it: vector instruction issue.  131 071 plans of 32 stages, M = 64 and 128: 3.8 ms ->
// 0.59 ms; 2^20 plans, M = 128: 14 -> 2.5 ms; 20 011 plans of 48 stages, M = 96: 4.1 -> 0.18 ms.  One
// lane per candidate with the durations in LDS (what this replaces, for up to 32 stages) held one
// wave per SIMD and issued 5 vector instructions and an LDS read per block update, and its check of
// an ordering read every pair of devices from memory; beyond 32 stages everything was 64-bit in LDS.
// Comparison schedules of 40 320 plans of 8 stages, M = 64: full-duplex channels 221 -> 30 us, GPipe's
// order 131 -> 34 us, transfers added to the stages 137 -> 22 us (64-bit in LDS before).
#include "pp_makespan.h"

#define SPLIT_NEG (-(1 << 30))

__device__ __forceinline__ int smax(int a, int b) { return a > b ? a : b; }

// u with the sign bit of `from`.
__device__ __forceinline__ int with_sign(int from, int u) { return (from & (int)0x80000000) | u; }

enum { SPLIT_FILL, SPLIT_FULL, SPLIT_DRAIN, SPLIT_BOTH };

// MODE: PP_SCHED_PE; PP_SCHED_DUPLEX: the two transfers of a channel (even places) do not wait for
// each other, so a channel's sides are idle from their own last items; PP_SCHED_ADDITIVE: the PE
// schedule of stages alone; PP_SCHED_GPIPE: see split_wave.
template <int RL, int KIND, int MODE>
__device__ __forceinline__ void split_sweep(int (&f)[RL], int (&b)[RL], int (&idle)[RL], const int (&df)[RL],
                                            const int (&db)[RL], int source, bool is_first, bool is_last) {
    int rf = __builtin_amdgcn_update_dpp(0, f[RL - 1], DPP_WAVE_SHR1, 0xf, 0xf, false);
    int rb = __builtin_amdgcn_update_dpp(0, b[0], DPP_WAVE_SHL1, 0xf, 0xf, false);
    rf = is_first ? source : rf;
    // forward side, downwards: f[i - 1] is still the previous sweep's
#pragma unroll
    for (int i = RL - 1; i >= 0; --i) {
        const int in = i ? f[i - 1] : rf;
        if (MODE == PP_SCHED_DUPLEX && !(i & 1)) {
            f[i] = with_sign(in, smax(f[i], in) + df[i]);
        } else if (KIND == SPLIT_FILL) {
            f[i] = smax(smax(f[i], b[i]), in) + df[i];
        } else if (KIND == SPLIT_FULL) {
            f[i] = smax(b[i], in) + df[i];
        } else if (KIND == SPLIT_DRAIN) {
            f[i] = with_sign(in, smax(b[i], in) + df[i]);
        } else {
            f[i] = with_sign(in, smax(idle[i], in) + df[i]);
            idle[i] = smax(idle[i], f[i]);
        }
    }
    rb = is_last ? f[RL - 1] : rb;
    // backward side, upwards: b[i + 1] is still the previous sweep's.  (The two sides of a channel do not
    // hold each other's values up under DUPLEX: marks can lie below -2^30 there, and an empty place must not
    // take its -2^30 from those.)
    constexpr int low = SPLIT_NEG;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
        const int in = i + 1 < RL ? b[i + 1 < RL ? i + 1 : i] : rb;
        if (MODE == PP_SCHED_DUPLEX && !(i & 1)) {
            b[i] = with_sign(in, smax(smax(b[i], in), low) + db[i]);
        } else if (KIND == SPLIT_FILL) {
            b[i] = with_sign(in, smax(f[i], in) + db[i]);
        } else if (KIND == SPLIT_FULL) {
            b[i] = smax(f[i], in) + db[i];
        } else if (KIND == SPLIT_DRAIN) {
            b[i] = smax(smax(b[i], f[i]), MODE == PP_SCHED_DUPLEX ? smax(in, low) : in) + db[i];
        } else {
            b[i] = with_sign(in, smax(idle[i], in) + db[i]);
            idle[i] = smax(idle[i], b[i]);
        }
    }
}

// GPipe's order: a forward wave over all microbatches, then a backward wave, each resource continuing
// from the end of its last forward item.  One sweep of one of them (a place whose input is negative
// has no item).
template <int RL, bool FORWARD>
__device__ __forceinline__ void split_wave(int (&x)[RL], int (&idle)[RL], const int (&d)[RL], int source, bool at_source) {
    int edge = FORWARD ? __builtin_amdgcn_update_dpp(0, x[RL - 1], DPP_WAVE_SHR1, 0xf, 0xf, false)
                       : __builtin_amdgcn_update_dpp(0, x[0], DPP_WAVE_SHL1, 0xf, 0xf, false);
    edge = at_source ? source : edge;
#pragma unroll
    for (int j = 0; j < RL; ++j) {
        const int i = FORWARD ? RL - 1 - j : j;
        const int in = FORWARD ? (i ? x[i ? i - 1 : 0] : edge) : (i + 1 < RL ? x[i + 1 < RL ? i + 1 : i] : edge);
        x[i] = with_sign(in, smax(idle[i], in) + d[i]);
        idle[i] = smax(idle[i], x[i]);
    }
}

// 64 candidates per workgroup of G waves, G = a.lanes_per.
template <int RL, int MODE>
__global__ __launch_bounds__(512) void k_makespan_split(mk_args a) {
    extern __shared__ int rows[];  // devices and bounds of 64 candidates, rows of SP; then 64 fault words
    // (with a header the data decide for the whole launch: k_makespan_lds does the others)
    if (!a.by_block) {
        unsigned long long vmax = a.hdr->pmax[threadIdx.x & (PP_PACK_BLOCKS - 1)];
        int mmax = 1;
        for (int q = 0; q < a.nM; ++q) mmax = a.Ms[q] > mmax ? a.Ms[q] : mmax;
        if (__ballot(!(vmax <= MK_SPLIT_CAP && mk_split_fits((long long)vmax, mmax, a.S)))) return;
    }
    // (resources: stages and channels, or stages alone)
    const int S = a.S, L = a.L, D = a.D, R = MODE == PP_SCHED_ADDITIVE ? S : 2 * S - 1, G = a.lanes_per, SP = S | 1;
    const int tid = threadIdx.x, T = blockDim.x;
    int *so = rows, *sb = rows + 64 * SP, *sf = sb + 64 * SP;
    const long long c0 = (long long)blockIdx.x * 64;
    for (int t = tid; t < 64 * S; t += T) {
        const int i = t / S, n = t - i * S;
        const long long c = c0 + i;
        int o = 0, e = 0;
        if (c < a.N) {
            if (a.orderings) o = a.orderings[c * a.ord_stride + n];
            e = a.bounds[c * a.bnd_stride + a.bnd_off + n];
        }
        so[i * SP + n] = o;
        sb[i * SP + n] = e;
    }
    __syncthreads();
    if (tid < 64) sf[tid] = c0 + tid < a.N ? mk_check_rows(a, c0 + tid, so + tid * SP, sb + tid * SP) : 0;
    __syncthreads();
    // lane q of candidate i holds the places q RL .. q RL + RL - 1 of G RL; place p is resource
    // p + 1 - pad.  RL is even and 2 S - 1 odd, so pad is odd: odd places are stages, even ones
    // channels.  (Stages alone: place p is stage p - pad.)
    const int lg = __builtin_ctz(G), i = tid >> lg, q = tid & (G - 1);
    const int pad = G * RL - R;
    const long long c = c0 + i;
    const bool live = c < a.N;
    const int fault = sf[i];
    const bool ok = live && !fault;
    const int *o = so + i * SP, *e = sb + i * SP;
    int df[RL], db[RL];
    long long worst = 0;
    auto stage = [&](int n, long long &x, long long &y) {
        const int e1 = e[n], e0 = n ? e[n - 1] : 0;
        x = a.PF[e1] - a.PF[e0];
        y = a.PB[e1] - a.PB[e0];
        worst = x + y > worst ? x + y : worst;
    };
    auto channel = [&](int n, long long &x, long long &y) {  // between stages n - 1 and n
        const size_t at = ((size_t)o[n - 1] * D + o[n]) * L + (size_t)(e[n - 1] - 1);
        x = a.XF[at];
        y = a.XB[at];
        worst = x + y > worst ? x + y : worst;
    };
#pragma unroll
    for (int k = 0; k < RL; ++k) {
        const int p = q * RL + k;
        long long x = 0, y = 0;
        bool empty = p < pad;
        if (MODE == PP_SCHED_ADDITIVE) {
            // the transfers over a stage's inbound link are part of its passes
            const int n = p - pad;
            if (ok && !empty) {
                stage(n, x, y);
                if (n) {
                    long long cx, cy;
                    channel(n, cx, cy);
                    x += cx;
                    y += cy;
                }
                worst = x + y > worst ? x + y : worst;
            }
            if (n == S - 1) { x += y; y = 0; }
        } else if (k & 1) {
            const int n = (p - pad) >> 1;
            if (ok && !empty) stage(n, x, y);
            if (n == S - 1 && MODE != PP_SCHED_GPIPE) { x += y; y = 0; }
        } else {
            const int n = (p + 1 - pad) >> 1;
            empty |= n < 1;
            if (ok && !empty) channel(n, x, y);
        }
        df[k] = (int)x;
        db[k] = empty ? SPLIT_NEG : (int)y;
    }
    for (int off = 1; off < G; off <<= 1) {
        const long long w = __shfl_xor(worst, off);
        worst = w > worst ? w : worst;
    }
    if (a.by_block) {
        int mmax = 1;
        for (int m = 0; m < a.nM; ++m) mmax = a.Ms[m] > mmax ? a.Ms[m] : mmax;
        // (GPipe's two waves take up to M + R - 1 of the largest forward and backward times each)
        const bool fits = !ok || mk_split_fits(worst, MODE == PP_SCHED_GPIPE ? 2ll * mmax + 4 * S : mmax, S);
        if (!__syncthreads_and(fits)) {
            if (live && q == 0) a.T_out[c * a.t_stride + a.t_off] = MK_NOT_TAKEN;
            return;
        }
    }
    const bool is_first = q == 0, is_last = q == G - 1;
    for (int m = 0; m < a.nM; ++m) {
        const int M = a.Ms[m], J = 2 * R - 1;
        int f[RL], b[RL], idle[RL];
#pragma unroll
        for (int k = 0; k < RL; ++k) f[k] = b[k] = SPLIT_NEG;
        if constexpr (MODE == PP_SCHED_GPIPE) {
#pragma unroll
            for (int k = 0; k < RL; ++k) idle[k] = 0;
            const int waves = M + R - 1 + pad;
            for (int t = 1; t <= waves; ++t) split_wave<RL, true>(f, idle, df, t <= M ? 0 : SPLIT_NEG, is_first);
            for (int t = 1; t <= waves - pad; ++t) split_wave<RL, false>(b, idle, db, t <= M ? 0 : SPLIT_NEG, is_last);
        } else {
        // sweeps: resource 1 serves microbatch m in sweep m + pad, its last backward item ends in
        // sweep M + J - 1 + pad; after sweep J + pad every resource has had a backward item
        const int full = J + pad, end = M + J - 1 + pad;
        int t = 1;
        for (; t <= full && t <= M; ++t) split_sweep<RL, SPLIT_FILL, MODE>(f, b, idle, df, db, 0, is_first, is_last);
        if (t <= full) {
#pragma unroll
            for (int k = 0; k < RL; ++k) idle[k] = smax(smax(f[k], b[k]), 0);
            for (; t <= full; ++t) split_sweep<RL, SPLIT_BOTH, MODE>(f, b, idle, df, db, SPLIT_NEG, is_first, is_last);
        }
        for (; t <= M; ++t) split_sweep<RL, SPLIT_FULL, MODE>(f, b, idle, df, db, 0, is_first, is_last);
        for (; t <= end; ++t) split_sweep<RL, SPLIT_DRAIN, MODE>(f, b, idle, df, db, SPLIT_NEG, is_first, is_last);
        }
        // resource 1 sits at place `pad`
        int Tv = 0;
#pragma unroll
        for (int k = 0; k < RL; ++k) Tv = q * RL + k == pad ? b[k] : Tv;
        if (live && q == pad / RL) {
            const int fq = fault;
            if (fq) pp_raise(a.status, fq);
            a.T_out[((long long)m * a.N + c) * a.t_stride + a.t_off] = fq ? PP_INF64 : (long long)Tv;
        }
    }
}

template <int RL>
static int launch_split(const mk_args &a, hipStream_t st) {
    const size_t lds = ((size_t)2 * 64 * (a.S | 1) + 64) * 4;
    const dim3 grid((unsigned)((a.N + 63) / 64)), block(64 * a.lanes_per);
    switch (a.variant) {
        case PP_SCHED_PE: hipLaunchKernelGGL((k_makespan_split<RL, PP_SCHED_PE>), grid, block, lds, st, a); break;
        case PP_SCHED_DUPLEX: hipLaunchKernelGGL((k_makespan_split<RL, PP_SCHED_DUPLEX>), grid, block, lds, st, a); break;
        case PP_SCHED_GPIPE: hipLaunchKernelGGL((k_makespan_split<RL, PP_SCHED_GPIPE>), grid, block, lds, st, a); break;
        case PP_SCHED_ADDITIVE: hipLaunchKernelGGL((k_makespan_split<RL, PP_SCHED_ADDITIVE>), grid, block, lds, st, a); break;
        default: return PP_ERR_INVALID_ARG;
    }
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}

int pp_launch_makespan_split(const mk_args &a, hipStream_t st) {
    // As few lanes per candidate as 32 places each allow (the two shifts per sweep are shared by
    // more resources), twice as many while the launch would leave SIMDs without a second wave.
    const int R = a.variant == PP_SCHED_ADDITIVE ? a.S : 2 * a.S - 1;
    mk_args b = a;
    int G = 1;
    while (G * 32 < R) G <<= 1;
    const long long groups = (a.N + 63) / 64;
    while (G < 8 && groups * G < 2048 && R > 14 * G) G <<= 1;
    b.lanes_per = G;
    const int RL = ((R + G - 1) / G + 3) & ~3;
    switch (RL) {
        case 4: case 8: return launch_split<8>(b, st);
        case 12: return launch_split<12>(b, st);
        case 16: return launch_split<16>(b, st);
        case 20: return launch_split<20>(b, st);
        case 24: return launch_split<24>(b, st);
        case 28: return launch_split<28>(b, st);
        case 32: return launch_split<32>(b, st);
    }
    return PP_ERR_INVALID_ARG;
}
