// Alg. 1 with channels that serve by readiness (PP_SCHED_FIFO), one lane per resource.
//
// Stages follow their lists, so a stage's next item is known and may be committed (start = the later
// of idle and ready) as soon as the preceding block has let its microbatch go, whatever the clock
// says elsewhere.  A channel takes, of its forward and its backward head, the one that was ready
// first (equal times: the earlier in list order), so it may commit a head once the other side's head
// is known too, or cannot be ready before or with it: every resource passes a lower bound of its
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
// What bounds it: instruction issue (about 75 vector and 85 scalar instructions per step, and 4.3
// items committed per candidate and step at 8 stages).  40 320 plans of 8 stages, M = 64: 9.35 ms (one
// lane per candidate, one item per step) -> 1.31 ms; with branches instead of combined conditions
// 1.52 ms.
#include "pp_makespan.h"

#define FIFO_THREADS 256

// LG = a.lanes_per lanes per candidate (a power of two, at least R), lane r - 1 is resource r.
__global__ __launch_bounds__(FIFO_THREADS) void k_makespan_fifo(mk_args a) {
    extern __shared__ int lds[];
    const int S = a.S, L = a.L, D = a.D, M = a.Ms[0], LG = a.lanes_per, SP = S | 1;
    const int R = 2 * S - 1, J = 2 * R - 1;
    const int tid = threadIdx.x, lane = tid & 63, per = FIFO_THREADS / LG;  // candidates per workgroup
    int Q = 1;
    while (Q < J) Q <<= 1;
    int *so = lds, *sb = so + per * SP, *sf = sb + per * SP, *left = sf + per, *rings = left + 1;
    const long long c0 = a.first + (long long)blockIdx.x * per;
    for (int t = tid; t < per * S; t += FIFO_THREADS) {
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
    if (tid == 0) *left = 0;
    __syncthreads();
    if (tid < per) sf[tid] = c0 + tid < a.N ? mk_check_rows(a, c0 + tid, so + tid * SP, sb + tid * SP) : 0;
    __syncthreads();
    const int i = tid / LG, r = tid - i * LG + 1;
    const long long c = c0 + i;
    const bool live = c < a.N, in = r <= R, stage = r & 1;
    const int fault = sf[i];
    // durations of the resource's forward and backward items
    int df = 0, db = 0;
    bool zero = false;
    long long sum = 0;
    if (live && !fault && in) {
        const int *o = so + i * SP, *e = sb + i * SP;
        const int n = r >> 1;  // stage n, or the channel between stages n - 1 and n
        long long x, y;
        if (stage) {
            const int e1 = e[n], e0 = n ? e[n - 1] : 0;
            x = a.PF[e1] - a.PF[e0];
            y = a.PB[e1] - a.PB[e0];
            if (n == S - 1) { x += y; y = 0; }
        } else {
            const size_t at = ((size_t)o[n - 1] * D + o[n]) * L + (size_t)(e[n - 1] - 1);
            x = a.XF[at];
            y = a.XB[at];
        }
        zero = x <= 0 || (y <= 0 && r < R);
        df = (int)x;
        db = (int)y;
        // (anything at 2^30 or above is out already: the sum of at most 63 such cannot overflow)
        x = x < MK_SPLIT_CAP ? x : MK_SPLIT_CAP;
        y = y < MK_SPLIT_CAP ? y : MK_SPLIT_CAP;
        sum = x + y;
    }
    int odd = zero;
    for (int off = 1; off < LG; off <<= 1) {
        sum += __shfl_xor(sum, off);
        odd |= __shfl_xor(odd, off);
    }
    // (the workgroup's candidates are taken or left together: k_makespan_variant simulates whole waves
    // of neighbours wherever one of them is left.  All four schedules, a seventh of the cuts with nothing to
    // send, 10^6 plans of 2 stages, M = 32: 1.95 ms plan by plan, 1.15 together, 1.19 in that kernel alone)
    if (live && !fault && (odd || sum > (long long)MK_SPLIT_CAP / M)) *left = 1;
    __syncthreads();
    const bool taken = *left == 0;
    bool running = live && !fault && taken;
    int *ring = rings + i * Q;  // when a microbatch left its last block (a microbatch is in one place)
    const int Qm = Q - 1, jb = 2 * R - r;
    // next forward and backward microbatch of the resource, when it is idle, bounds for its neighbours
    int nf = 1, nb = 1, idle = 0, outF = 0, outB = 0;
    const unsigned long long group = (LG == 64 ? ~0ull : (1ull << LG) - 1) << (lane & ~(LG - 1));
    const bool isFirst = r == 1, isLast = r == R, channel = in & !stage;
    const int bias = jb - r;  // forward item nf comes before backward item nb in list order iff nf - nb <= bias
    // (every step commits at least one item of every candidate that is not through; conditions are
    // combined with & and |, without branches)
    for (long long step = 0; step <= (long long)J * M && __builtin_amdgcn_ballot_w64(running); ++step) {
        const int slotF = ring[nf & Qm], slotB = ring[nb & Qm];
        const int nfL = __builtin_amdgcn_update_dpp(0, nf, DPP_WAVE_SHR1, 0xf, 0xf, false);
        const int nbR = __builtin_amdgcn_update_dpp(0, isLast ? nf : nb, DPP_WAVE_SHL1, 0xf, 0xf, false);
        const int lbL = __builtin_amdgcn_update_dpp(0, outF, DPP_WAVE_SHR1, 0xf, 0xf, false);
        const int lbR = __builtin_amdgcn_update_dpp(0, isLast ? outF : outB, DPP_WAVE_SHL1, 0xf, 0xf, false);
        const bool hasF = nf <= M, hasB = !isLast & (nb <= M);
        const bool atF = hasF & (isFirst | (nfL > nf)), atB = hasB & (nbR > nb);
        // when the heads are ready, or no earlier than
        int rF = atF ? slotF : lbL;
        rF = isFirst ? 0 : rF;
        const int rB = atB ? slotB : lbR;
        const bool listF = nf - nb <= bias;  // the forward head comes first in list order
        const bool stageF = hasF & (!hasB | listF);
        const bool soonerF = (rF < rB) | ((rF == rB) & listF);
        const bool pickF = stage ? stageF : (atF & (!atB | soonerF));
        const bool sureF = atB | !hasB | (rB > rF), sureB = !hasF | (rF > rB);
        bool can = stage ? ((stageF & atF) | (!stageF & atB)) : ((atF & sureF) | (!atF & atB & sureB));
        can = can & in & running;
        const unsigned long long who = __builtin_amdgcn_ballot_w64(can);
        const bool stuck = running & !(who & group);
        if (__builtin_amdgcn_ballot_w64(stuck)) {
            // some candidate waits everywhere: its channel head with the earliest start
            const bool head = stuck & channel & (atF | atB);
            const int ready = atF ? rF : rB;
            int first = head ? (ready > idle ? ready : idle) : INT32_MAX;
            const int mine = first;
            for (int off = 1; off < LG; off <<= 1) {
                const int o = __shfl_xor(first, off);
                first = o < first ? o : first;
            }
            const unsigned long long at = __builtin_amdgcn_ballot_w64(head & (mine == first)) & group;
            can = can | (head & (at != 0) & (lane == (int)__builtin_ctzll(at | 1ull << 63)));
        }
        const int begin = pickF ? rF : rB, m = pickF ? nf : nb;
        const int end = (begin > idle ? begin : idle) + (pickF ? df : db);
        if (can) ring[m & Qm] = end;
        idle = can ? end : idle;
        nf += can & pickF;
        nb += can & !pickF;
        // no later item of the resource can end before these (a stage whose next item is the other
        // side's has to serve that first)
        const bool nextF = (nf <= M) & (isLast | (nb > M) | (nf - nb <= bias));
        outF = (rF > idle ? rF : idle) + df + ((stage & !nextF) ? db : 0);
        outB = (rB > idle ? rB : idle) + db + ((stage & nextF) ? df : 0);
        // through when stage 0 has served its last item
        const unsigned long long through = __builtin_amdgcn_ballot_w64(isFirst & ((isLast ? nf : nb) > M));
        running = running & !(through & group);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (live && r == 1) {
        if (fault) pp_raise(a.status, fault);
        a.T_out[c] = fault ? PP_INF64 : (taken ? (long long)idle : MK_NOT_TAKEN);
    }
}

int pp_launch_makespan_fifo(const mk_args &a, hipStream_t st) {
    const int R = 2 * a.S - 1, J = 2 * R - 1;
    if (R > 64) return PP_ERR_INVALID_ARG;
    mk_args b = a;
    b.lanes_per = 1;
    while (b.lanes_per < R) b.lanes_per <<= 1;
    int Q = 1;
    while (Q < J) Q <<= 1;
    const int per = FIFO_THREADS / b.lanes_per;
    const size_t lds = ((size_t)per * (2 * (a.S | 1) + 1 + Q) + 1) * 4;
    // A launch has fewer than 2^32 threads.  At up to 64 lanes per candidate that is fewer candidates than
    // a list may hold (all 12! orderings, 32 lanes each), so long lists take several launches.
    const long long groups = (a.N + per - 1) / per, most = ((1ll << 32) - 1) / FIFO_THREADS;
    for (long long g = 0; g < groups; g += most) {
        b.first = g * per;
        hipLaunchKernelGGL(k_makespan_fifo, dim3((unsigned)(groups - g < most ? groups - g : most)), dim3(FIFO_THREADS), lds, st, b);
        if (hipGetLastError() != hipSuccess) return PP_ERR_HIP;
    }
    return PP_OK;
}
