// Makespan (Eq. 2) of plans with replicated stages, S <= 16.
#include "pp_makespan.h"
#include "pp_makespan_sweep.h"

__device__ __forceinline__ long long ceil_div64(long long x, long long y) { return x / y + (x % y != 0); }

// Plans with replicated stages (Sec. III-B): stage s runs on reps[s] GPUs of consecutive ranks,
// a replica takes ceil(p / k) per microbatch, a transfer between stages of k' and k replicas
// ceil(d / (k' k min b)) with the minimum over the links between the two GPU sets, and a
// replicated stage ends with a ring AllReduce of ceil(2 (k-1) sum alpha / (k min b)) (Eq. 1)
// that starts when its last backward pass has finished.  T is the later of the last backward
// block on stage 0 and the end of the last AllReduce (Eq. 2).  One lane per candidate; the
// plan with S stages of candidate c is read from the triangular arrays.
template <int S>
__device__ __forceinline__ void rep_body(const mk_args &a) {
    constexpr int R = 2 * S - 1, J = 4 * S - 3;
    constexpr int t_off = S - 1, bnd_off = S * (S - 1) / 2;
    const int lane = threadIdx.x, L = a.L, D = a.D;
    const long long c = (long long)blockIdx.x * 64 + lane;
    const bool live = c < a.N;
    const int M = a.Ms[0];
    long long dur[J + 1], A[S];
    long long worst = 0, amax = 0;
    int fault = 0;
    const bool none = live && a.W[c * a.t_stride + t_off] == PP_INF64;  // no plan with S stages
    const bool work = live && !none;
    const int *bd = a.bounds + c * a.bnd_stride + bnd_off;
    const int *rp = a.reps + c * a.bnd_stride + bnd_off;
    const int *o = a.orderings + c * a.ord_stride;
    if (work) {
        int prev = 0, used = 0;
        for (int s = 0; s < S; ++s) {
            int e = bd[s], k = rp[s];
            if (e <= prev || e > L || k < 1 || k > D) fault |= PP_FAULT_BOUNDS;
            prev = e;
            used += k;
        }
        if (prev != L || used != D) fault |= PP_FAULT_BOUNDS;
        for (int n = 0; n < D; ++n) {
            int d = o[n];
            bool bad = d < 0 || d >= D;
            for (int q = 0; q < n; ++q) bad |= (o[q] == d);
            if (bad) fault |= PP_FAULT_ORDERING;
        }
    }
    const bool ok = work && !fault;
    int e0 = 0, n = 0, kprev = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        long long F = 0, Bk = 0, cf = 0, cb = 0, As = 0;
        if (ok) {
            const int e = bd[s], k = rp[s];
            F = ceil_div64(a.PF[e] - a.PF[e0], k);
            Bk = ceil_div64(a.PB[e] - a.PB[e0], k);
            if (k > 1) {
                long long m = PP_INF64;
                for (int u = n; u < n + k; ++u)
                    for (int v = n; v < n + k; ++v)
                        if (u != v) {
                            long long x = a.bw[(size_t)o[u] * D + o[v]];
                            m = x < m ? x : m;
                        }
                As = ceil_div64(2 * (long long)(k - 1) * (a.PA[e] - a.PA[e0]), (long long)k * m);
            }
            if (s) {
                long long mf = PP_INF64, mb = PP_INF64;
                for (int u = n - kprev; u < n; ++u)
                    for (int v = n; v < n + k; ++v) {
                        long long x = a.bw[(size_t)o[u] * D + o[v]], y = a.bw[(size_t)o[v] * D + o[u]];
                        mf = x < mf ? x : mf;
                        mb = y < mb ? y : mb;
                    }
                cf = ceil_div64(a.actf[e0 - 1], (long long)kprev * k * mf);
                cb = ceil_div64(a.actb[e0 - 1], (long long)kprev * k * mb);
            }
            e0 = e;
            n += k;
            kprev = k;
        }
        A[s] = As;
        amax = As > amax ? As : amax;
        long long w = F + Bk > cf + cb ? F + Bk : cf + cb;
        worst = w > worst ? w : worst;
        const int r = 2 * s + 1;
        if (s == S - 1) {
            dur[R] = F + Bk;
        } else {
            dur[r] = F;
            dur[2 * R - r] = Bk;
        }
        if (s) {
            dur[r - 1] = cf;
            dur[2 * R - (r - 1)] = cb;
        }
    }
    dur[0] = 0;
    if (ok) {
        fault |= overflow_fault(worst, M, S);
        if (amax >= PP_CAP62 / 2) fault |= PP_FAULT_OVERFLOW;
    }
    // the later of the last backward block on stage 0 and the end of every AllReduce
    auto finish = [&](auto &fin) {
        long long T = (long long)fin[J];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int jb = s == S - 1 ? R : 2 * R - (2 * s + 1);
            const long long t = (long long)fin[jb] + A[s];
            T = (A[s] > 0 && t > T) ? t : T;
        }
        return T;
    };
    const bool narrow = !ok || fault || worst <= (long long)0x7fffffff / ((long long)M + 4 * S - 4);
    long long T;
    if (__all(narrow)) T = sweep_regs<S, int>(dur, M, finish);
    else T = sweep_regs<S, long long>(dur, M, finish);
    if (live) {
        if (fault) pp_raise(a.status, fault);
        a.T_out[c * a.t_stride + t_off] = (none || fault) ? PP_INF64 : T;
    }
}

// All stage counts of a call in one launch, blockIdx.y = 0 for the largest (the longest) first:
// a wave's schedule is one chain of dependent instructions, and a launch per stage count left most
// of the chip idle for as long as that chain takes, D times over.  SMAX: the registers of the
// largest body are those of the launch, so it is not larger than D needs by more than 3.
// Bound by that chain.  8 stage counts of 40320 candidates: 8 launches of 28 us -> 134 us; 12 of
// 3001 candidates: 12 of 45 us -> 61 us; a whole call with L = 26, D = 6: 237 -> 151 us.
template <int S>
__device__ __forceinline__ void rep_pick(const mk_args &a, int xi) {
    if (xi == S) rep_body<S>(a);
    else if constexpr (S > 1) rep_pick<S - 1>(a, xi);
}
template <int SMAX>
__global__ __launch_bounds__(64) void k_rep_makespan(mk_args a) {
    rep_pick<SMAX>(a, a.D - (int)blockIdx.y);
}

int mk_launch_replicated(const mk_args &a, hipStream_t st) {
    const dim3 grid((unsigned)((a.N + 63) / 64), a.D), block(64);
    if (a.D <= 4) hipLaunchKernelGGL(k_rep_makespan<4>, grid, block, 0, st, a);
    else if (a.D <= 8) hipLaunchKernelGGL(k_rep_makespan<8>, grid, block, 0, st, a);
    else if (a.D <= 12) hipLaunchKernelGGL(k_rep_makespan<12>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(k_rep_makespan<16>, grid, block, 0, st, a);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
