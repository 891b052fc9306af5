// The sweeps of a schedule of at most 16 stages with the state of a lane's candidate in registers
// (the recurrence: pp_makespan.hip), for k_makespan_regs and k_rep_makespan.
#pragma once

#include "pp_common.h"

// med3(old, fresh, sel) for 0 <= old <= fresh < 2^31: fresh if the scalar sel is all ones, old if it is 0.
__device__ __forceinline__ int keep_or_take(int old, int fresh, unsigned sel) {
    int r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(old), "v"(fresh), "s"(sel));
    return r;
}
__device__ __forceinline__ long long keep_or_take(long long old, long long fresh, unsigned sel) {
    return sel ? fresh : old;
}

// One sweep restricted to blocks LO..HI (compile-time), no validity tests.
template <int S, typename V, int LO, int HI>
__device__ __forceinline__ void sweep_blocks(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1]) {
    constexpr int R = 2 * S - 1, J = 2 * R - 1;
    const V finR_prev = fin[R];
    // forward blocks and the merged block R, descending so that fin[j-1] is still the
    // previous sweep's value
#pragma unroll
    for (int j = R; j >= 1; --j) {
        if (j < LO || j > HI) continue;
        V idle = fin[j] > fin[2 * R - j] ? fin[j] : fin[2 * R - j];
        V ready = j > 1 ? fin[j - 1] : (V)0;
        fin[j] = (idle > ready ? idle : ready) + dur[j];
    }
    // backward blocks: the resource may just have been used by this sweep's forward block
#pragma unroll
    for (int j = J; j >= R + 1; --j) {
        if (j < LO || j > HI) continue;
        V idle = fin[j] > fin[2 * R - j] ? fin[j] : fin[2 * R - j];
        V ready = j == R + 1 ? finR_prev : fin[j - 1];
        fin[j] = (idle > ready ? idle : ready) + dur[j];
    }
}

template <int S, typename V, int T>
__device__ __forceinline__ void ramp_up(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1]) {
    if constexpr (T <= 4 * S - 4) {
        sweep_blocks<S, V, 1, T>(fin, dur);
        ramp_up<S, V, T + 1>(fin, dur);
    }
}

template <int S, typename V, int U>
__device__ __forceinline__ void ramp_down(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1]) {
    if constexpr (U <= 4 * S - 4) {
        sweep_blocks<S, V, U + 1, 4 * S - 3>(fin, dur);
        ramp_down<S, V, U + 1>(fin, dur);
    }
}

// All M + 4S - 4 sweeps with the finish times in registers; returns the finish of the last
// backward block on stage 0.  Block j works in sweep t iff t-M+1 <= j <= t.  When the
// pipeline fills completely (M >= J-1) the sweeps split into a ramp-up (blocks 1..t), a
// steady phase (all blocks) and a ramp-down (blocks t-M+1..J) whose block ranges are known at
// compile time.  A shorter pipeline still has such a ramp-up (its first M sweeps) and ramp-down
// (its last M-1); in the sweeps between them, and in every sweep for S > 8 (where unrolling
// every sweep would be too much code), every block is computed and the update is kept or
// dropped by a select: with 32-bit times a median of three against a per-block scalar that is
// 0 or all ones (finish times never decrease, so med3(old, new, ~0) = new and
// med3(old, new, 0) = old), with 64-bit times a per-lane compare.
// `result(fin)` turns the final finish times into the value returned.
// Sweep t with every block computed and the update of the blocks outside [t-M+1, t] dropped.
template <int S, typename V>
__device__ __forceinline__ void sweep_selected(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1], int t, int M) {
    constexpr int R = 2 * S - 1, J = 2 * R - 1;
    const V finR_prev = fin[R];
    if constexpr (sizeof(V) == 4) {
        // bit j of `act`: block j works in this sweep
        const int jlo = t - M + 1 > 1 ? t - M + 1 : 1, jhi = t < J ? t : J;
        const unsigned long long act = ((2ull << jhi) - 1) & ~((1ull << jlo) - 1);
        // groups of G blocks without an active one are skipped altogether
        constexpr int G = 5;
#pragma unroll
        for (int jh = R; jh >= 1; jh -= G) {
            const int jl = jh - G + 1 > 1 ? jh - G + 1 : 1;
            if (!(act & (((2ull << jh) - 1) & ~((1ull << jl) - 1)))) continue;
#pragma unroll
            for (int j = jh; j >= jl; --j) {
                V idle = fin[j] > fin[2 * R - j] ? fin[j] : fin[2 * R - j];
                V ready = j > 1 ? fin[j - 1] : (V)0;
                V nv = (idle > ready ? idle : ready) + dur[j];
                fin[j] = keep_or_take(fin[j], nv, (act >> j) & 1 ? ~0u : 0u);
            }
        }
#pragma unroll
        for (int jh = J; jh >= R + 1; jh -= G) {
            const int jl = jh - G + 1 > R + 1 ? jh - G + 1 : R + 1;
            if (!(act & (((2ull << jh) - 1) & ~((1ull << jl) - 1)))) continue;
#pragma unroll
            for (int j = jh; j >= jl; --j) {
                V idle = fin[j] > fin[2 * R - j] ? fin[j] : fin[2 * R - j];
                V ready = j == R + 1 ? finR_prev : fin[j - 1];
                V nv = (idle > ready ? idle : ready) + dur[j];
                fin[j] = keep_or_take(fin[j], nv, (act >> j) & 1 ? ~0u : 0u);
            }
        }
    } else {
        // j is in [t-M+1, t] iff (unsigned)(j - (t-M+1)) <= M-1; kept in a vector register so
        // that the tests run on the vector unit next to the arithmetic
        const unsigned width = (unsigned)(M - 1);
        int jlo = t - M + 1;
        asm volatile("" : "+v"(jlo));
#pragma unroll
        for (int j = R; j >= 1; --j) {
            V idle = fin[j] > fin[2 * R - j] ? fin[j] : fin[2 * R - j];
            V ready = j > 1 ? fin[j - 1] : (V)0;
            V nv = (idle > ready ? idle : ready) + dur[j];
            fin[j] = (unsigned)(j - jlo) <= width ? nv : fin[j];
        }
#pragma unroll
        for (int j = J; j >= R + 1; --j) {
            V idle = fin[j] > fin[2 * R - j] ? fin[j] : fin[2 * R - j];
            V ready = j == R + 1 ? finR_prev : fin[j - 1];
            V nv = (idle > ready ? idle : ready) + dur[j];
            fin[j] = (unsigned)(j - jlo) <= width ? nv : fin[j];
        }
    }
}

// The first M sweeps of a pipeline that never fills (M <= J-2): blocks 1..t.
template <int S, typename V, int T>
__device__ __forceinline__ void ramp_up_to(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1], int M) {
    if constexpr (T <= 4 * S - 5) {
        if (T > M) return;
        sweep_blocks<S, V, 1, T>(fin, dur);
        ramp_up_to<S, V, T + 1>(fin, dur, M);
    }
}

// The last sweeps of a pipeline, blocks U+1..J for every U+1 >= lo.
template <int S, typename V, int U>
__device__ __forceinline__ void ramp_down_from(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1], int lo) {
    if constexpr (U <= 4 * S - 4) {
        if (U + 1 >= lo) sweep_blocks<S, V, U + 1, 4 * S - 3>(fin, dur);
        ramp_down_from<S, V, U + 1>(fin, dur, lo);
    }
}

// Sweeps M+1..J of a pipeline that never fills, for a microbatch count known at compile time:
// the window of M blocks moves up by one block per sweep.
template <int S, typename V, int M, int T>
__device__ __forceinline__ void slide_window(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1]) {
    if constexpr (T <= 4 * S - 3) {
        sweep_blocks<S, V, T - M + 1, T>(fin, dur);
        slide_window<S, V, M, T + 1>(fin, dur);
    }
}

// Picks the instance of slide_window for the run-time microbatch count m (1 <= m <= J-2).
template <int S, typename V, int M>
__device__ __forceinline__ void slide_window_for(V (&fin)[4 * S - 3 + 1], const V (&dur)[4 * S - 3 + 1], int m) {
    if constexpr (M <= 4 * S - 5) {
        if (m == M) {
            slide_window<S, V, M, M + 1>(fin, dur);
            return;
        }
        slide_window_for<S, V, M + 1>(fin, dur, m);
    }
}

template <int S, typename V, typename Result>
__device__ __forceinline__ long long sweep_regs(const long long (&dur64)[4 * S - 3 + 1], int M, Result result) {
    constexpr int R = 2 * S - 1, J = 2 * R - 1;
    V dur[J + 1], fin[J + 1];
#pragma unroll
    for (int j = 1; j <= J; ++j) { dur[j] = (V)dur64[j]; fin[j] = 0; }
    dur[0] = fin[0] = 0;
    if constexpr (S <= 8) {
        if (M >= J - 1) {
            ramp_up<S, V, 1>(fin, dur);
            for (int t = J; t <= M; ++t) sweep_blocks<S, V, 1, J>(fin, dur);
            ramp_down<S, V, 1>(fin, dur);
        } else {
            ramp_up_to<S, V, 1>(fin, dur, M);                                   // sweeps 1..M
            if constexpr (sizeof(V) == 4) slide_window_for<S, V, 1>(fin, dur, M);       // sweeps M+1..J
            else for (int t = M + 1; t <= J; ++t) sweep_selected<S, V>(fin, dur, t, M);
            ramp_down_from<S, V, 1>(fin, dur, J - M + 2);                       // sweeps J+1..J+M-1
        }
        return result(fin);
    }
    const int sweeps = M + 2 * R - 2;
    for (int t = 1; t <= sweeps; ++t) sweep_selected<S, V>(fin, dur, t, M);
    return result(fin);
}
