// Alg. 1 with channels that serve by readiness (PP_SCHED_FIFO), resources over lanes.
//
// Stages follow their lists, so a stage's next item is known and may be committed (start = the later
// of idle and ready) as soon as the preceding block has let its microbatch go, whatever the clock
// says elsewhere.  A channel takes, of its forward and its backward head, the one that was ready
// first (equal times: the earlier in list order), so it may commit a head once the other side's head
// is known too, or cannot be ready before it: every resource passes a lower bound of its
// next finish time to its neighbours (its idle time or bounds passed to it, plus durations).  With
// positive durations this is the schedule of the event simulation in k_makespan_variant, which
// commits the item with the earliest start next: all items that are ready by a start are committed
// before it there.  All resources that can commit do so in the same step, so a candidate takes about
// as many steps as its pipeline has sweeps instead of one per item; if none can, the earliest start
// among the waiting channel heads is next (equal starts: the lowest resource), as in the simulation.
//
// Left to k_makespan_variant (marked MK_NOT_TAKEN), with the rest of their workgroup: zero durations, whose order within one point in
// time only the simulation defines, and times whose sum does not fit 30 bits (no schedule that
// always has an item in service is longer than the sum of all items).
//
// Four neighbouring resources share a lane and are looked at one after the other, upwards in one pass and downwards
// in the next, so that an item can go through several resources in a pass: 8 stages, M = 64 take about 205 passes,
// where looking at all resources at once takes 265 (eight a lane 180, but with them a launch of 40 000 plans has one
// wave per SIMD).
//
// What bounds it: instruction issue, vector units busy 87 % of the time (about 55 instructions look at a resource: which head is next, when it can be
// served, and the bounds for the neighbours).  40 320 plans of 8 stages, M = 64: 9.35 ms (one lane per candidate, one item per
// step), 1.31 ms (one lane per resource, all at once), 0.28 ms now.
#include "pp_makespan.h"

#define FIFO_THREADS 256   // a workgroup's threads, about one per resource, for the loads; its first wave goes on
#define FIFO_RL 4          // resources per lane; even places are stages, odd ones channels
#define FIFO_LATE (1 << 30)  // later than any time

struct fifo_lane {
    // per resource: next forward and backward microbatch, when it is idle, no later item of a side ends before,
    // durations, and forward item nf comes before backward item nb in list order iff nf <= nb + bias
    int nf[FIFO_RL], nb[FIFO_RL], idle[FIFO_RL], outF[FIFO_RL], outB[FIFO_RL], df[FIFO_RL], db[FIFO_RL], bias[FIFO_RL];
    bool last[FIFO_RL];   // the merged block: its items are forward items, and what resource R - 1 takes backward
    bool nextF[FIFO_RL];  // stages: the next item is a forward one
    // what the resource looked at before in this pass has served: its end, and which side (last: both)
    int end;
    bool didF, didB;
    int M, Qm;
    int *ring;  // when a microbatch left its last block (a microbatch is in one place)
    bool first;
};

// Resource K of the lane, in a pass upwards (UP) or downwards: the neighbour looked at before in this pass is as it
// is now, the other as it was before the pass.  nfL, lowL: the left neighbour's next forward microbatch and bound;
// nbR, lowR: the right one's; atF, atB: what the ring said, before the pass, of the resource's heads.
template <int K, bool UP>
__device__ __forceinline__ bool fifo_step(fifo_lane &s, int nfL, int lowL, int nbR, int lowR, int slotF, int slotB) {
    constexpr bool stage = !(K & 1);
    const int nf = s.nf[K], nb = s.nb[K];
    // (the head is what the neighbour has let go just now)
    if (UP && K > 0) slotF = s.didF && nfL == nf + 1 ? s.end : slotF;
    if (!UP && K + 1 < FIFO_RL) slotB = s.didB && nbR == nb + 1 ? s.end : slotB;
    // when the heads are ready, or no earlier than
    const bool atF = nfL > nf, atB = nbR > nb;
    int rF = atF ? slotF : lowL, rB = atB ? slotB : lowR;
    if (K == 0) rF = s.first ? 0 : rF;
    bool pickF;
    if (stage) {
        pickF = s.nextF[K];
    } else {
        // the head that is ready first, if its side is the one that has it
        rF = nf <= s.M ? rF : FIFO_LATE;
        rB = nb <= s.M ? rB : FIFO_LATE;
        pickF = rF < rB + (nf <= nb + s.bias[K] ? 1 : 0);
    }
    const bool doF = atF & pickF, doB = atB & !pickF, can = doF | doB;
    const int m = pickF ? nf : nb, ready = pickF ? rF : rB;
    const int end = (ready > s.idle[K] ? ready : s.idle[K]) + (pickF ? s.df[K] : s.db[K]);
    if (can) s.ring[m & s.Qm] = end;
    s.end = end;
    s.didF = doF;
    s.didB = stage ? doB | (doF & s.last[K]) : doB;
    s.idle[K] = can ? end : s.idle[K];
    s.nf[K] = nf + doF;
    s.nb[K] = nb + s.didB;
    // No later item of the resource can end before these.  A stage whose next item is one side's has to serve that
    // before the other side's, from when that one's head can be there on: a channel that holds the stage's next
    // forward item thereby knows that nothing comes back before it.  (With the idle time alone in that place a
    // candidate of 8 stages, M = 64, waited everywhere 26 times and took up to 660 passes instead of 260.)
    int outF = (rF > s.idle[K] ? rF : s.idle[K]) + s.df[K], outB = (rB > s.idle[K] ? rB : s.idle[K]) + s.db[K];
    if (stage) {
        const int most = s.nb[K] + s.bias[K];
        const bool nextF = s.nextF[K] = s.nf[K] <= (most < s.M ? most : s.M);
        const int thenF = (rF > outB ? rF : outB) + s.df[K], thenB = (rB > outF ? rB : outF) + s.db[K];
        outF = nextF ? outF : thenF;
        outB = nextF ? thenB : outB;
        outB = s.last[K] ? outF : outB;
    }
    s.outF[K] = outF;
    s.outB[K] = outB;
    return can;
}

// One pass over the lane's resources; returns whether an item was committed.
template <bool UP>
__device__ __forceinline__ bool fifo_pass(fifo_lane &s) {
    constexpr int E = FIFO_RL - 1;
    int slotF[FIFO_RL], slotB[FIFO_RL];
#pragma unroll
    for (int k = 0; k < FIFO_RL; ++k) {
        slotF[k] = s.ring[s.nf[k] & s.Qm];
        slotB[k] = s.ring[s.nb[k] & s.Qm];
    }
    int nfL = __builtin_amdgcn_update_dpp(0, s.nf[E], DPP_WAVE_SHR1, 0xf, 0xf, false);
    int lowL = __builtin_amdgcn_update_dpp(0, s.outF[E], DPP_WAVE_SHR1, 0xf, 0xf, false);
    const int nbR = __builtin_amdgcn_update_dpp(0, s.nb[0], DPP_WAVE_SHL1, 0xf, 0xf, false);
    const int lowR = __builtin_amdgcn_update_dpp(0, s.outB[0], DPP_WAVE_SHL1, 0xf, 0xf, false);
    nfL = s.first ? s.M + 1 : nfL;  // (the source has every microbatch)
    bool any = false;
    static_assert(FIFO_RL == 4, "");
    if (UP) {
        any |= fifo_step<0, UP>(s, nfL, lowL, s.nb[1], s.outB[1], slotF[0], slotB[0]);
        any |= fifo_step<1, UP>(s, s.nf[0], s.outF[0], s.nb[2], s.outB[2], slotF[1], slotB[1]);
        any |= fifo_step<2, UP>(s, s.nf[1], s.outF[1], s.nb[3], s.outB[3], slotF[2], slotB[2]);
        any |= fifo_step<3, UP>(s, s.nf[2], s.outF[2], nbR, lowR, slotF[3], slotB[3]);
    } else {
        any |= fifo_step<3, UP>(s, s.nf[2], s.outF[2], nbR, lowR, slotF[3], slotB[3]);
        any |= fifo_step<2, UP>(s, s.nf[1], s.outF[1], s.nb[3], s.outB[3], slotF[2], slotB[2]);
        any |= fifo_step<1, UP>(s, s.nf[0], s.outF[0], s.nb[2], s.outB[2], slotF[1], slotB[1]);
        any |= fifo_step<0, UP>(s, nfL, lowL, s.nb[1], s.outB[1], slotF[0], slotB[0]);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return any;
}

// LG = a.lanes_per lanes per candidate (a power of two, at least R / 4), place p = 4 (lane) + k is resource p + 1.
__global__ __launch_bounds__(FIFO_THREADS) void k_makespan_fifo(mk_args a) {
    extern __shared__ int lds[];
    const int S = a.S, L = a.L, D = a.D, M = a.Ms[0], LG = a.lanes_per, SP = S | 1;
    const int R = 2 * S - 1, J = 2 * R - 1;
    const int tid = threadIdx.x, lane = tid & 63, per = 64 / LG;  // candidates per workgroup
    int Q = 1;
    while (Q < J) Q <<= 1;
    // (rings an odd number of words apart: their slots lie in different banks)
    int *so = lds, *sb = so + per * SP, *sf = sb + per * SP, *rings = sf + per;
    const long long c0 = a.first + (long long)blockIdx.x * per;
    for (int t = tid; t < per * S; t += blockDim.x) {
        const int i = t / S, n = t - i * S;
        const long long c = c0 + i;
        int o = 0, e = 0;
        if (c < a.N) {
            if (a.orderings) o = a.orderings[c * S + n];
            e = a.bounds[c * S + n];
        }
        so[i * SP + n] = o;
        sb[i * SP + n] = e;
    }
    __syncthreads();
    if (tid < per) sf[tid] = c0 + tid < a.N ? mk_check_rows(a, c0 + tid, so + tid * SP, sb + tid * SP) : 0;
    __syncthreads();
    if (tid >= 64) return;
    const int i = lane / LG, q = lane - i * LG;
    const long long c = c0 + i;
    const bool live = c < a.N;
    const int fault = sf[i];
    const bool ok = live && !fault;
    fifo_lane s;
    s.M = M;
    s.Qm = Q - 1;
    s.ring = rings + i * (Q + 1);
    s.first = q == 0;
    bool zero = false;
    long long sum = 0;
#pragma unroll
    for (int k = 0; k < FIFO_RL; ++k) {
        const int r = q * FIFO_RL + k + 1;
        long long x = 0, y = 0;
        if (ok && r <= R) {
            const int *o = so + i * SP, *e = sb + i * SP;
            const int n = r >> 1;  // stage n, or the channel between stages n - 1 and n
            if (!(k & 1)) {
                const int e1 = e[n], e0 = n ? e[n - 1] : 0;
                x = a.PF[e1] - a.PF[e0];
                y = a.PB[e1] - a.PB[e0];
                if (n == S - 1) { x += y; y = 0; }
            } else {
                const size_t at = ((size_t)o[n - 1] * D + o[n]) * L + (size_t)(e[n - 1] - 1);
                x = a.XF[at];
                y = a.XB[at];
            }
            zero |= x <= 0 || (y <= 0 && r < R);
        }
        s.df[k] = (int)x;
        s.db[k] = (int)y;
        // (anything at 2^30 or above is out already: the sum of at most 126 such cannot overflow)
        x = x < MK_SPLIT_CAP ? x : MK_SPLIT_CAP;
        y = y < MK_SPLIT_CAP ? y : MK_SPLIT_CAP;
        sum += x + y;
        s.last[k] = r == R;
        s.bias[k] = 2 * (R - r);
        // (places beyond the last resource, and candidates that are not simulated, have no items)
        s.nf[k] = s.nb[k] = ok && r <= R ? 1 : M + 1;
        s.nextF[k] = s.nf[k] <= M;  // (the first item of every resource)
        s.idle[k] = s.outF[k] = s.outB[k] = 0;
    }
    int odd = zero;
    for (int off = 1; off < LG; off <<= 1) {
        sum += __shfl_xor(sum, off);
        odd |= __shfl_xor(odd, off);
    }
    // (the workgroup's candidates are taken or left together: k_makespan_variant simulates whole waves
    // of neighbours wherever one of them is left.  All four schedules, a seventh of the cuts with nothing to
    // send, 10^6 plans of 2 stages, M = 32: 1.95 ms plan by plan, 1.15 together, 1.19 in that kernel alone)
    const bool taken = !__builtin_amdgcn_ballot_w64(ok && (odd || sum > (long long)MK_SPLIT_CAP / M));
    const unsigned long long group = (LG == 64 ? ~0ull : (1ull << LG) - 1) << (lane & ~(LG - 1));
    // (every step commits at least one item of every candidate that is not through)
    for (long long step = 0; taken && step <= (long long)J * M; ++step) {
        const bool running = s.first && s.nb[0] <= M;
        const unsigned long long run = __builtin_amdgcn_ballot_w64(running);
        if (!run) break;
        const bool up = fifo_pass<true>(s), down = fifo_pass<false>(s);
        const unsigned long long who = __builtin_amdgcn_ballot_w64(up | down);
        const bool stuck = (run & group) && !(who & group);
        if (!__builtin_amdgcn_ballot_w64(stuck)) continue;
        // some candidate waits everywhere: its channel head with the earliest start (equal: the lowest resource)
        const int nbR = __builtin_amdgcn_update_dpp(0, s.nb[0], DPP_WAVE_SHL1, 0xf, 0xf, false);
        int best = INT32_MAX, which = 0, ready[FIFO_RL], m[FIFO_RL];
        bool forth[FIFO_RL];
#pragma unroll
        for (int k = 1; k < FIFO_RL; k += 2) {
            const int right = k + 1 < FIFO_RL ? s.nb[k + 1 < FIFO_RL ? k + 1 : k] : nbR;
            const bool atF = s.nf[k - 1] > s.nf[k], atB = right > s.nb[k];
            forth[k] = atF;
            m[k] = atF ? s.nf[k] : s.nb[k];
            ready[k] = s.ring[m[k] & s.Qm];
            const int begin = ready[k] > s.idle[k] ? ready[k] : s.idle[k];
            if (stuck && (atF | atB) && begin < best) { best = begin; which = k; }
        }
        const int mine = best;
        for (int off = 1; off < LG; off <<= 1) {
            const int o = __shfl_xor(best, off);
            best = o < best ? o : best;
        }
        const unsigned long long at = __builtin_amdgcn_ballot_w64(which != 0 && mine == best) & group;
        const bool go = which != 0 && at && lane == (int)__builtin_ctzll(at | 1ull << 63);
#pragma unroll
        for (int k = 1; k < FIFO_RL; k += 2) {
            if (!go || which != k) continue;
            const int end = best + (forth[k] ? s.df[k] : s.db[k]);
            s.ring[m[k] & s.Qm] = end;
            s.idle[k] = end;
            if (forth[k]) ++s.nf[k];
            else ++s.nb[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (live && q == 0) {
        if (fault) pp_raise(a.status, fault);
        a.T_out[c] = fault ? PP_INF64 : (taken ? (long long)s.idle[0] : MK_NOT_TAKEN);
    }
}

int pp_launch_makespan_fifo(const mk_args &a, hipStream_t st) {
    const int R = 2 * a.S - 1, J = 2 * R - 1;
    if (R > 64) return PP_ERR_INVALID_ARG;
    mk_args b = a;
    b.lanes_per = 1;
    while (b.lanes_per * FIFO_RL < R) b.lanes_per <<= 1;
    int Q = 1;
    while (Q < J) Q <<= 1;
    const int per = 64 / b.lanes_per;
    const size_t lds = (size_t)per * (2 * (a.S | 1) + 1 + Q + 1) * 4;
    int each = 1;  // (threads per candidate: its resources, rounded up to a power of two)
    while (each < R) each <<= 1;
    const int threads = per * each;
    // A launch has fewer than 2^32 threads.  At up to 64 threads per candidate that is fewer candidates than
    // a list may hold (all 12! orderings, 32 each), so long lists take several launches.
    const long long groups = (a.N + per - 1) / per, most = ((1ll << 32) - 1) / threads;
    for (long long g = 0; g < groups; g += most) {
        b.first = g * per;
        hipLaunchKernelGGL(k_makespan_fifo, dim3((unsigned)(groups - g < most ? groups - g : most)), dim3(threads), lds, st, b);
        if (hipGetLastError() != hipSuccess) return PP_ERR_HIP;
    }
    return PP_OK;
}
