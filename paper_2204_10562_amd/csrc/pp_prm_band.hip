// Plans with replicated stages (PRM, Alg. 4; recursion for W(l, xi, r, i) in Sec. IV-B, see pp_prm.hip) from the
// few cells of every state that a plan as good as the best can use.
//
// A stage of layers of p in all on k GPUs takes at least M p / k, so W(l, xi, r, i) >= M P[l] / i, and the stages
// that follow take at least M (P[L] - P[l]) / (D - i) on the other GPUs.  Let V be a time that no best plan of
// three stages or more exceeds, whatever the ordering.  Then only the cells l with M P[l] <= V i and
// M (P[L] - P[l]) <= V (D - i) can lie on one, and by induction the recursion over those alone has the true value and
// the true first minimiser (l', r') wherever the value is at most V.
// V comes from one plan per number of stages with every link as slow as the slowest of the cluster: no best plan of
// any ordering is slower.  (Plans of two stages have a bound and cuts of their own: their first stage needs no table.)
// 8 GPUs, 128 layers: 5 cells of 128 in a state; 12 GPUs in servers of 4, 75 layers of uneven times: 19 of 75.  Where a
// band is wider than two cells per lane, and with int64 values, k_prm does the launch.
//
// 8 or 16 lanes per candidate, one per cell, so that a wave has eight or four candidates; wider bands in two parts, and
// only those states that are wide.  The states on i GPUs by ascending i.  For each (r, i) the minima over r' of every
// cut come first, for all numbers of stages at once.  Where the channels are hidden behind the stages, as they nearly always are
// (what follows from the work before and after a cut bounds every value from below), these are the minima over the last
// stage's replicas that the states have left behind; else the channel term of every cut and r' is worked out and the states
// on i - r GPUs are read from the wave's scratch memory.  They go to LDS by cut, and are then read for every cell with the
// cut's last stage, again for all numbers of stages.  The GPUs' bandwidth minima are taken from the ordering as they
// are needed: lane u holds the minimum over the links of rank u, which grow by a rank at a time, and a suffix minimum over
// the lanes gives all r'.  With few candidates the waves of a workgroup share them, each with its part of the r of every i.
//
// What bounds it: trips to the scratch memory, which the waves in flight (2.5 per SIMD) spread over more than the caches hold,
// and instructions.  All 40320 orderings of 8 GPUs, 128 layers: 3.80 ms with k_prm, 0.275 with every channel term and
// every minimum over r', 0.196 now; 3001 orderings of 12 GPUs, 75 layers: 1.95, 0.226, 0.173 ms.  (Plans were read back with
// the minima over their links worked out again and a trip to memory per r' tried: 30 % of the first one's time.)
#include "pp_prm.h"
#include "pp_dp_row.h"

#define PRM_PREP_THREADS 1024
#define PRM_TRIES 16      // times that are tried for a bound
#define PRM_TRY_CELLS 36  // the largest gives bands of about so many cells: few more than are of use

// One workgroup: input checks, prefix sums, whether int32 values do (all as in k_prm, which reports what is wrong
// if it is), the bounds, the bands, and M (QF + QB) with the one-hot remainders per (r, l).  A chain of short steps:
// 26 us with 8 GPUs, 33 with 12, of which the times that are tried take 11 and 18 (55 with a search that halves the
// range, double sums and 32 tries: LDS reads at random are what the sixteen waves wait for).
__global__ __launch_bounds__(PRM_PREP_THREADS) void k_prm_prep(prm_args a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_bad;
    __shared__ unsigned long long s_af, s_ab, s_lo, s_hi;
    __shared__ double s_bound[17];
    __shared__ unsigned s_fits[17];
    __shared__ int s_reach[3][17][PRM_TRIES], s_pair[136];
    __shared__ float2 s_each[17];
    const int L = a.L, D = a.D, L1 = L + 1, tid = threadIdx.x, T = PRM_PREP_THREADS, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long M = a.M;
    long long *PF = (long long *)smem, *PB = PF + L1, *PA = PB + L1;
    float2 *PT = (float2 *)(PA + L1);  // [l] work and AllReduce bytes of the layers before
    float *act = (float *)(PT + L1);  // [l] bytes over the cut after l layers, both ways
    if (tid == 0) { s_bad = 0; s_af = s_ab = s_hi = 0; s_lo = ~0ull; a.band[PRM_BAND_PARTS] = 0; }
    __syncthreads();
    {
        bool bad = L < D || D < 2;
        unsigned long long af = 0, ab = 0, lo = ~0ull, hi = 0;
        for (int l = tid; l < L; l += T) {
            const long long x = a.fwd[l], y = a.bwd[l], z = a.alpha[l];
            const long long f = a.actf[l], b = a.actb[l];
            bad |= x < 0 || y < 0 || z < 0 || x >= PP_CAP62 || y >= PP_CAP62 || z >= PP_CAP62;
            if (l + 1 < L) {
                bad |= f < 0 || b < 0;
                af = (unsigned long long)f > af ? (unsigned long long)f : af;
                ab = (unsigned long long)b > ab ? (unsigned long long)b : ab;
            }
            PF[l + 1] = x; PB[l + 1] = y; PA[l + 1] = z;
            act[l + 1] = l + 1 < L ? (float)f + (float)b : 0.0f;
        }
        for (int t = tid; t < D * D; t += T)
            if (t / D != t % D) {
                const long long b = a.bw[t];
                bad |= b <= 0;
                lo = (unsigned long long)b < lo ? (unsigned long long)b : lo;
                hi = (unsigned long long)b > hi ? (unsigned long long)b : hi;
            }
        if (tid == 0) { PF[0] = PB[0] = PA[0] = 0; act[0] = 0.0f; }
        if (tid <= 16) { s_bound[tid] = 0.0; s_fits[tid] = 0; }
        if (bad) s_bad = 1;
        // (the waves that read something)
        if (wave * 64 < L || wave * 64 < D * D) {
            for (int off = 32; off; off >>= 1) {
                const unsigned long long x = __shfl_xor(af, off), y = __shfl_xor(ab, off), z = __shfl_xor(hi, off), u = __shfl_xor(lo, off);
                af = x > af ? x : af;
                ab = y > ab ? y : ab;
                hi = z > hi ? z : hi;
                lo = u < lo ? u : lo;
            }
            if (lane == 0) {
                atomicMax(&s_af, af);
                atomicMax(&s_ab, ab);
                atomicMax(&s_hi, hi);
                atomicMin(&s_lo, lo);
            }
        }
    }
    __syncthreads();
    if (s_bad) return;
    if (wave < 3) {
        // one wave per array: neighbours of L / 64 entries per lane
        long long *P = wave == 0 ? PF : wave == 1 ? PB : PA;
        const int each = (L + 63) / 64, first = 1 + lane * each, end = first + each < L1 ? first + each : L1;
        unsigned long long sum = 0;
        bool big = false;
        for (int l = first; l < end; ++l) sum += (unsigned long long)P[l];
        big |= sum >= (unsigned long long)PP_CAP62;
        unsigned long long before = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned long long o = (unsigned long long)__shfl_up((long long)before, off);
            before += lane >= off ? o : 0;
        }
        big |= before >= (unsigned long long)PP_CAP62;
        before -= sum;
        for (int l = first; l < end; ++l) {
            before += (unsigned long long)P[l];
            big |= before >= (unsigned long long)PP_CAP62;
            P[l] = (long long)before;
        }
        if (big) s_bad = 1;
    }
    __syncthreads();
    if (s_bad) return;
    // (the same conditions as in k_prm)
    const long long f = PF[L], b = PB[L], al = PA[L], lim = 1ll << 30, bmin = (long long)s_lo;
    const unsigned long long exact = 1ull << 53;
    const bool narrow = f + b < PP_CAP62 / (M + 4 * D) && al < PP_CAP62 / (2 * D) && M < (1 << 20) && (long long)s_hi < lim / D &&
                        cdiv64((long long)s_af, bmin) + cdiv64((long long)s_ab, bmin) < lim / M && 2 * al / bmin + 1 < lim / 2 &&
                        f + b + 2 < lim / (2 * M) && s_af < exact && s_ab < exact && (unsigned long long)al < exact / (2 * D);
    if (!narrow) return;
    for (int l = tid; l <= L; l += T) {
        a.pre_out[l] = PF[l];
        a.pre_out[L1 + l] = PB[l];
        a.pre_out[2 * L1 + l] = PA[l];
        PT[l] = make_float2((float)(PF[l] + PB[l]), (float)PA[l]);
    }
    int2 *ut = (int2 *)(a.band + PRM_BAND_HDR);
    for (int t = tid; t < D * L1; t += T) {
        const int r = t / L1 + 1, l = t - (r - 1) * L1;
        const unsigned pf = (unsigned)PF[l], pb = (unsigned)PB[l], qf = pf / (unsigned)r, qb = pb / (unsigned)r;
        ut[t] = make_int2((int)(M * (long long)(qf + qb)), (1 << (int)(pf - qf * r)) | (1 << (16 + (int)(pb - qb * r))));
    }
    // ---- bounds: for PRM_TRIES times, the last cell that i GPUs reach in xi stages within it (and the replicas of the
    // last stage), by ascending xi.  Each is a plan; that it is not always the best only costs cells.  (In float: a
    // difference of prefix sums is off by 2^-23 of the whole, which is taken off the time here with what the difference
    // itself adds, and the few roundings of the size of the time, below 2^-20, are added in the end.)
    const double Md = (double)M, ideal = Md * (double)(f + b) / D, fixed = 2.0 * Md + 1.0;
    const float slow = (float)(Md / (double)bmin);
    auto trial = [&](int k) {
        const float x = (float)(k + 1) / PRM_TRIES;
        return ideal * (1.0 + (double)((float)PRM_TRY_CELLS / L * x * __builtin_sqrtf(x))) + 2.0 * fixed;
    };
    const int k = tid & (PRM_TRIES - 1);
    const float v = (float)(trial(k) - fixed);  // (ceil adds less than `fixed` to a stage or transfer)
    // Bands are narrow only if there is a plan of D stages within the largest of the times tried.  That has one GPU a
    // stage: where the layers between two neighbours of the cuts that can be had over the slowest link take longer, there
    // is none, and k_prm does the launch (unless bands of all cells will do).  (The last wave; one link slower by 1000:
    // 342 us without bands, 351; 374 with the whole look, 200 orderings of 8 GPUs, 128 layers; 861, 869; 903, 300 of 12, 75.)
    if (wave == T / 64 - 1 && L > prm_band_cells(D, 16) + 1) {
        const float most = __shfl(v, PRM_TRIES - 1);
        int before = 0;  // the last cut of the chunks done, or 0 (0 and L are ends of stages, too)
        bool none = false;
        for (int l0 = 1; l0 <= L; l0 += 64) {
            const int l = l0 + lane;
            const bool cut = l == L || (l < L && slow * act[l] <= most);
            const unsigned long long cuts = __ballot(cut), lower = cuts & ((1ull << lane) - 1);
            const int prev = lower ? l0 + 63 - __builtin_clzll(lower) : before;
            if (cut) none |= Md * (double)(PF[l] - PF[prev] + PB[l] - PB[prev]) > (double)most * (1.0 + 0x1p-20);
            before = cuts ? l0 + 63 - __builtin_clzll(cuts) : before;
        }
        if (none) s_bad = 1;
    }
    for (int t = tid; t < 3 * 17 * PRM_TRIES; t += T) ((int *)s_reach)[t] = 0;
    if (tid < D * (D + 1) / 2) {
        // (GPUs before, replicas) by descending GPUs before
        int q = 1;
        while (q * (q + 1) / 2 <= tid) ++q;
        s_pair[tid] = (D - q) << 8 | (tid - q * (q - 1) / 2 + 1);
    }
    if (tid >= 1 && tid <= D) s_each[tid] = make_float2((float)(Md / tid), (float)(2.0 * (tid - 1) / tid / (double)bmin));
    __syncthreads();
    if (s_bad) return;
    int far = 1;  // the largest power of four below L
    while (far * 4 < L) far *= 4;
    int now = 0;
    for (int xi = 1; xi <= D; ++xi) {
        const int next = now == 2 ? 0 : now + 1;
        int(*from)[PRM_TRIES] = s_reach[now], (*to)[PRM_TRIES] = s_reach[next], *idle = s_reach[next == 2 ? 0 : next + 1][0];
        for (int t = tid; t < 17 * PRM_TRIES; t += T) idle[t] = 0;
        // of the pairs, those with at least xi - 1 GPUs before
        const int pairs = xi == 1 ? D : (D - xi + 1) * (D - xi + 2) / 2;
        for (int p = tid / PRM_TRIES; p < pairs; p += T / PRM_TRIES) {
            const int pair = xi == 1 ? p + 1 : s_pair[p], before = pair >> 8, r = pair & 0xff;
            const int at = xi == 1 ? 0 : from[before][k], c = at >> 8, i = before + r;
            if (xi > 1 && (c == 0 || slow * act[c] > v * (float)((at & 0xff) * r))) continue;
            const float2 e = s_each[r], pc = PT[c], all = PT[L];
            const float vr = v - 0x1p-21f * (e.x * all.x + e.y * all.y);
            if (i == D) {
                if (e.x * (all.x - pc.x) + e.y * (all.y - pc.y) <= vr && c < L) atomicOr(&s_fits[xi], 1u << k);
                continue;
            }
            int lo = c;  // the last cell that fits: three looked at a time
            for (int step = far; step; step >>= 2) {
                const int l1 = lo + step, l2 = l1 + step, l3 = l2 + step;
                const float2 p1 = PT[l1 < L ? l1 : L], p2 = PT[l2 < L ? l2 : L], p3 = PT[l3 < L ? l3 : L];
                lo = l1 < L && e.x * (p1.x - pc.x) + e.y * (p1.y - pc.y) <= vr ? l1 : lo;
                lo = l2 < L && e.x * (p2.x - pc.x) + e.y * (p2.y - pc.y) <= vr ? l2 : lo;
                lo = l3 < L && e.x * (p3.x - pc.x) + e.y * (p3.y - pc.y) <= vr ? l3 : lo;
            }
            // (a cut whose transfers fit, if the next stage has as many replicas)
            while (lo > c && slow * act[lo] > v * (float)(r * r)) --lo;
            if (lo > c) atomicMax(&to[i][k], lo << 8 | r);
        }
        now = next;
        __syncthreads();
    }
    if (tid >= 2 && tid <= D && s_fits[tid])
        // (the first time that fits)
        s_bound[tid] = trial(__builtin_ctz(s_fits[tid])) * (1.0 + 1e-5) + 1.0;
    __syncthreads();
    // ---- bands, of all cells where there is no bound
    if (tid < 64) {
        const int i = lane & 31, two = lane >> 5;
        long long V = 0;
        for (int xi = two ? 2 : 3; xi <= (two ? 2 : D); ++xi) {
            const long long x = s_bound[xi] > 0.0 && s_bound[xi] < (double)lim ? (long long)s_bound[xi] : lim;
            V = x > V ? x : V;
        }
        int w = 0;
        if (i >= 1 && i < D) {
            // first l >= 1 from which the rest fits, last l < L up to which i GPUs do
            int lo = 1, hi = L;
            while (lo < hi) {
                const int l = (lo + hi) >> 1;
                if (M * (f + b - PF[l] - PB[l]) <= V * (D - i)) hi = l;
                else lo = l + 1;
            }
            int c = 0, e = L - 1;
            while (c < e) {
                const int l = (c + e + 1) >> 1;
                if (M * (PF[l] + PB[l]) <= V * i) c = l;
                else e = l - 1;
            }
            w = c - lo + 1 > 0 ? c - lo + 1 : 0;
            a.band[(two ? PRM_BAND_LO2 : PRM_BAND_LO) + i] = lo;
            a.band[(two ? PRM_BAND_W2 : PRM_BAND_W) + i] = w;
        }
        int widest = two ? 0 : w;
        for (int off = 32; off; off >>= 1) widest = row_imax(widest, __shfl_xor(widest, off));
        const int lanes = D <= 8 && widest <= prm_band_cells(D, 8) ? 8 : 16;
        if (tid == 0) {
            a.band[PRM_BAND_LANES] = lanes;
            a.band[PRM_BAND_PARTS] = widest > prm_band_cells(D, 16) ? 0 : widest > lanes ? (widest + lanes - 1) / lanes : 1;
        }
    }
}

// Minimum over a candidate's lanes (all of them get it), and over its lanes from each one on (t: the lane's place).
template <int LANES>
__device__ __forceinline__ int row_min(int v) {
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, true));   // quad_perm:[1,0,3,2]
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, true));   // quad_perm:[2,3,0,1]
    v = row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, true));  // row_half_mirror
    return LANES == 8 ? v : row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, true));  // row_mirror
}
template <int LANES>
__device__ __forceinline__ int row_suffix_min(int v, int t) {
    int x = __builtin_amdgcn_update_dpp(v, v, 0x101, 0xf, 0xf, false);  // row_shl:1 (of 16 lanes)
    v = LANES == 16 || t < 7 ? row_imin(v, x) : v;
    x = __builtin_amdgcn_update_dpp(v, v, 0x102, 0xf, 0xf, false);
    v = LANES == 16 || t < 6 ? row_imin(v, x) : v;
    x = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xf, 0xf, false);
    v = LANES == 16 || t < 4 ? row_imin(v, x) : v;
    return LANES == 8 ? v : row_imin(v, __builtin_amdgcn_update_dpp(v, v, 0x108, 0xf, 0xf, false));
}

#define PRM_BAND_HIDDEN 0x8000  // with a cut: no r' before it has channels that matter (L < 2^15)

struct prm_rec { int u, ra, oh; };  // M (QF + QB) + QA, remainder of the AllReduce quotient, one-hot remainders

template <int LANES>
struct prm_band_wave {
    int D, M, L1, t;     // t: the lane's place among its candidate's
    const int2 *ut;      // [D][L1]
    const double *PA, *AF, *AB;
    const int *bw;       // [D][D]
    const int *o;        // [LANES] the candidate's devices
    __device__ __forceinline__ prm_rec rec(int r, int l, double den, double inv) const {
        const int2 x = ut[(r - 1) * L1 + l];
        prm_rec q = {x.x, 0, x.y};
        if (r > 1) q.u += prm_floor_div(2.0 * (r - 1) * PA[l], den, inv, q.ra);
        return q;
    }
    // the last stage [l', l): M (F + B) + A
    __device__ __forceinline__ int last(const prm_rec &q, const prm_rec &ql) const {
        const int flags = __popc((unsigned)(q.oh & (ql.oh - 0x10001)));
        return ql.u - q.u + (int)__mul24(flags, M) + (ql.ra > q.ra);
    }
    __device__ __forceinline__ int channel(int l, int rr, int mf, int mb) const {
        const double f = (double)rr * (double)mf, b = (double)rr * (double)mb;
        return M * (prm_ceil_div(AF[l], f, prm_inv(f)) + prm_ceil_div(AB[l], b, prm_inv(b)));
    }
};

// LDS: the workgroup's tables, which no candidate changes, and what a wave has for itself.
struct prm_band_lds {
    const double *PA, *AF, *AB;
    const int2 *ut;
    const int *bw, *band;
    int4 *rows;  // [candidate of the wave][cells] records of the cuts
    int *gs;     // [candidate of the wave][cells][prm_band_row] Gmin by cut and stages before
    int *os;     // [64] devices
    int *best;   // [3][64], one for the workgroup: the best plans of another wave
};

// TEAM: the waves of the workgroup share candidates, each with its part of the r of every i.  STAGES: a multiple of 4, and no
// state has more stages before its last.
template <int LANES, bool TEAM, int STAGES>
__device__ __forceinline__ void prm_band_run(const prm_args &a, const prm_band_lds &lds, int wave, int waves, int wib, int team) {
    constexpr int EACH = 64 / LANES;  // candidates of a wave
    const int L = a.L, D = a.D, L1 = L + 1, lane = threadIdx.x & 63, t = lane & (LANES - 1), group = lane - t;
    const int tri = D * (D + 1) / 2;
    const int *band = lds.band;
    auto number = [&](int k) { return __builtin_amdgcn_readfirstlane(band[k]); };
    const int parts = number(PRM_BAND_PARTS);
    const unsigned NS64 = (unsigned)prm_states(D - 1) * 64;
    int *Wt = (int *)(a.scratch + (size_t)wave * parts * prm_band_slot_bytes(D));  // [part][state][64]
    unsigned short *At = (unsigned short *)(Wt + (size_t)NS64 * parts);            // the cut, and PRM_BAND_HIDDEN
    int *Gt = (int *)(At + (size_t)NS64 * parts);                                  // [part][GPUs, stages][64]
    int *In = Gt + (size_t)(D * (D - 1) / 2) * 64 * parts;  // [GPUs i][64] minima over the links between the ranks from one on up to i
    const int gsize = D * (D - 1) / 2 * 64;
    int4 *rows = lds.rows + group / LANES * prm_band_cells(D, LANES);
    const int ROW = prm_band_row(D);
    int *gs = lds.gs + group / LANES * prm_band_cells(D, LANES) * ROW;
    prm_band_wave<LANES> w;
    w.D = D; w.M = a.M; w.L1 = L1; w.t = t;
    w.ut = lds.ut; w.PA = lds.PA; w.AF = lds.AF; w.AB = lds.AB; w.bw = lds.bw;
    w.o = lds.os + group;
    const int INF = PP_INF32;
    const prm_rec none = {0, 0, 0x10001};  // nothing before the first layer
    // the wave that has r: its work falls with r, so there and back over the waves
    auto turn_of = [&](int r) {
        const int turn = (r - 1) / team, at = (r - 1) - turn * team;
        return turn & 1 ? team - 1 - at : at;
    };
    for (long long part = wave; part * EACH < a.N; part += waves) {
        const long long c = part * EACH + group / LANES;
        const bool have = c < a.N;
        // ---- ordering (a bad one is reported, and planned as 0, 1, 2, .. for nobody)
        int d = have && t < D ? a.ord[c * D + t] : t;
        bool wrong = t < D && (d < 0 || d >= D);
        row_lds_sync();
        lds.os[lane] = d;
        row_lds_sync();
        for (int q = 0; q < D; ++q) wrong |= q < t && t < D && w.o[q] == d;
        const bool bad = (__ballot(wrong) >> group & ((1ull << LANES) - 1)) != 0;
        d = bad || t >= D ? (t < D ? t : 0) : d;
        row_lds_sync();
        lds.os[lane] = d;
        row_lds_sync();
        // the minima over r begin above everything.  (Of a team, other waves first touch them for two GPUs, behind a barrier; that
        // of one GPU is stored.)
        for (int k = TEAM ? wib : 0; k < parts * (gsize / 64); k += TEAM ? team : 1)
            if (k % (gsize / 64)) Gt[k * 64 + lane] = INF;
        // ---- states by ascending number of GPUs; i == D: cell L alone, lane xi - 1 keeps the best r
        int wbest = INF, rbest = 0, lbest = 0;  // (lbest: the cut, and PRM_BAND_HIDDEN)
        const int ou = w.o[t];
        int inner = INF;  // of the links between rank t and those after it, both ways
        int whole = INF;  // of those between the first t ranks
        for (int i = 1; i <= D; ++i) {
            const bool top = i == D;
            // the links of rank i - 1 join: from rank t on, the minimum over the pairs of ranks t .. i - 1
            const int on = w.o[i - 1];
            inner = t < i - 1 ? row_imin(inner, row_imin(w.bw[ou * D + on], w.bw[on * D + ou])) : INF;
            const int inside = row_suffix_min<LANES>(inner, t), first_i = __shfl(inside, group);
            whole = t == i ? first_i : whole;
            if (!TEAM || wib == 0) In[(unsigned)i * 64 + lane] = inside;
            int out_f = INF, out_b = INF;  // of the links between rank t and the last r ranks, there and back
            const int lo = top ? L : number(PRM_BAND_LO + i), wd = top ? 1 : number(PRM_BAND_W + i);
            const float least = (float)lds.ut[lo].x / (float)i * 0.9999f;  // (see hidden)
            for (int r = 1; r <= i; ++r) {
                const int n0 = i - r;  // GPUs of the sub-problem
                const int od = w.o[n0];
                out_f = row_imin(out_f, w.bw[ou * D + od]);
                out_b = row_imin(out_b, w.bw[od * D + ou]);
                if (TEAM && turn_of(r) != wib) continue;
                // r times the minimum over the ordered pairs of the last stage's ranks
                const int links = __shfl(inside, group + n0);
                const double den = r < 2 ? 1.0 : (double)r * (double)links, inv = prm_inv(den);
                if (n0 == 0) {
                    for (int c0 = 0; c0 < wd; c0 += LANES) {
                        const int v = w.last(none, w.rec(r, row_imin(lo + c0 + t, L), den, inv));
                        if (top) {
                            if (t == 0) { wbest = v; rbest = D; }
                        } else if (c0 + t < wd) {
                            Wt[(unsigned)(c0 / LANES) * NS64 + prm_sid(i, 1, i) * 64 + lane] = v;
                            if (i == 1) Gt[(c0 / LANES) * gsize + lane] = v;
                            else atomicMin(Gt + (c0 / LANES) * gsize + i * (i - 1) / 2 * 64 + lane, v);
                        }
                    }
                    continue;
                }
                const int lo_p = number(PRM_BAND_LO + n0), w_p = number(PRM_BAND_W + n0);
                const prm_rec qL = top ? w.rec(r, L, den, inv) : none;
                // from rank t on to the last r ranks, both ways
                const int mf = row_suffix_min<LANES>(t < n0 ? out_f : INF, t), mb = row_suffix_min<LANES>(t < n0 ? out_b : INF, t);
                if (top) {
                    // two stages: any cut, the first stage on all n0 GPUs
                    const int links0 = __shfl(whole, group + n0);
                    const double den0 = n0 < 2 ? 1.0 : (double)n0 * (double)links0, inv0 = prm_inv(den0);
                    const int f0 = __shfl(mf, group), b0 = __shfl(mb, group);  // (from rank 0 on: r' = n0)
                    const int lo2 = number(PRM_BAND_LO2 + n0), w2 = number(PRM_BAND_W2 + n0);
                    int best = INF, at = 0;
                    for (int j = 0; j < w2; j += LANES) {
                        const int k = row_imin(lo2 + j + t, L - 1);
                        const int first = w.last(none, w.rec(n0, k, den0, inv0)), x = w.channel(k, n0 * r, f0, b0);
                        const int y = w.last(w.rec(r, k, den, inv), qL);
                        const int v = row_imax(row_imax(first, x), y);
                        if (j + t < w2 && v < best) { best = v; at = k; }
                    }
                    const int m = row_min<LANES>(best), k = row_min<LANES>(best == m ? at : INF);
                    if (t == 1 && m < wbest) { wbest = m; rbest = r; lbest = k; }
                    if (n0 < 2) continue;  // (three stages need two GPUs before the last)
                }
                // Gmin of every cut and number of stages: over r' of max(W(l', xi - 1, r', n0), X[r']).  Where no X[r'] of
                // any cut is more than any value of these states can be (M P[l] / i, which follows from the work before and
                // after the cut; ut for one replica is M times the work before it), max with it changes no value, and the minima
                // over r' are there already.  (In float, with room for its roundings and the two quotients'.)
                const float most = (float)a.M * __int_as_float(band[PRM_BAND_MOST + n0]) / ((float)((n0 - t) * r) * (float)row_imin(mf, mb));
                const bool hidden = !__ballot(t < n0 && !(most * 1.0001f + (float)(2 * a.M) < least));
                row_lds_sync();
                for (int c0 = 0; c0 < w_p; c0 += LANES) {
                    const int lp = row_imin(lo_p + c0 + t, L);  // the lane's cut
                    const bool cut = c0 + t < w_p;
                    const prm_rec qp = w.rec(r, lp, den, inv);
                    if (cut) rows[c0 + t] = make_int4(qp.u, qp.ra, qp.oh, top ? w.last(qp, qL) : 0);
                    const int *Wp = Wt + (unsigned)(c0 / LANES) * NS64 + prm_sid(n0, 1, 1) * 64;
                    // (a block of four numbers of stages to the wave's LDS; a number has cuts from itself on)
                    auto leave = [&](int s, int g0, int g1, int g2, int g3) {
                        if (cut)
                            *(int4 *)(gs + (c0 + t) * ROW + s) =
                                make_int4(lp > s ? g0 : INF, lp > s + 1 ? g1 : INF, lp > s + 2 ? g2 : INF, lp > s + 3 ? g3 : INF);
                    };
                    if (hidden) {
                        // (past the L1 cache: atomics leave them in the next one)
                        const int *Gp = Gt + (c0 / LANES) * gsize + n0 * (n0 - 1) / 2 * 64;
                        int g[STAGES];
#pragma unroll
                        for (int s = 0; s < STAGES; ++s)
                            g[s] = s < n0 ? __hip_atomic_load(Gp + s * 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : INF;
#pragma unroll
                        for (int s = 0; s < STAGES; s += 4)
                            if (s < n0) leave(s, g[s], g[s + 1], g[s + 2], g[s + 3]);
                        continue;
                    }
                    int g[STAGES];  // [xi - 2]
#pragma unroll
                    for (int s = 0; s < STAGES; ++s) g[s] = INF;
#pragma unroll 1
                    for (int rp = 1; rp <= n0; ++rp) {
                        const int x = w.channel(lp, rp * r, __shfl(mf, group + n0 - rp), __shfl(mb, group + n0 - rp));
                        // (the states of s + 1 stages on n0 GPUs begin at that of one replica; one stage has all n0)
                        int v[STAGES];
#pragma unroll
                        for (int s = 0; s < STAGES; s += 4) {
                            if (s > n0 - rp) continue;
                            // (of a block, also what belongs to the states after these: not used)
                            v[s] = Wp[(s * (n0 + 1) - s * (s + 1) / 2 + rp - 1) * 64 + lane];
                            v[s + 1] = Wp[((s + 1) * (n0 + 1) - (s + 1) * (s + 2) / 2 + rp - 1) * 64 + lane];
                            v[s + 2] = Wp[((s + 2) * (n0 + 1) - (s + 2) * (s + 3) / 2 + rp - 1) * 64 + lane];
                            v[s + 3] = Wp[((s + 3) * (n0 + 1) - (s + 3) * (s + 4) / 2 + rp - 1) * 64 + lane];
                        }
#pragma unroll
                        for (int s = 0; s < STAGES; s += 4) {
                            if (s > n0 - rp) continue;
                            if (s) g[s] = row_imin(g[s], row_imax(v[s], x));
                            else if (rp == n0) g[0] = row_imax(v[0], x);
                            if (s + 1 <= n0 - rp) g[s + 1] = row_imin(g[s + 1], row_imax(v[s + 1], x));
                            if (s + 2 <= n0 - rp) g[s + 2] = row_imin(g[s + 2], row_imax(v[s + 2], x));
                            if (s + 3 <= n0 - rp) g[s + 3] = row_imin(g[s + 3], row_imax(v[s + 3], x));
                        }
                    }
#pragma unroll
                    for (int s = 0; s < STAGES; s += 4)
                        if (s < n0) leave(s, g[s], g[s + 1], g[s + 2], g[s + 3]);
                }
                row_lds_sync();
                if (top) {
                    // lane xi - 1 looks at the cuts for xi stages
                    const bool on = t >= 2 && t <= n0;
                    int best = INF, at = 0;
                    for (int j = 0; j < w_p; ++j) {
                        const int v = row_imax(gs[j * ROW + (on ? t - 1 : 0)], rows[j].w);
                        at = v < best ? lo_p + j : at;
                        best = row_imin(v, best);
                    }
                    if (on && best < wbest) { wbest = best; rbest = r; lbest = hidden ? at | PRM_BAND_HIDDEN : at; }
                    continue;
                }
                // every cell of the states: the best cut
                for (int c0 = 0; c0 < wd; c0 += LANES) {
                    const int l = row_imin(lo + c0 + t, L);  // the lane's cell
                    const prm_rec ql = w.rec(r, l, den, inv);
                    int best[STAGES], at[STAGES];
#pragma unroll
                    for (int s = 0; s < STAGES; ++s) { best[s] = INF; at[s] = 0; }
#pragma unroll 1
                    for (int j = 0; j < w_p; ++j) {
                        const int4 q = rows[j];
                        const prm_rec qj = {q.x, q.y, q.z};
                        const int last = lo_p + j < l ? w.last(qj, ql) : INF;
#pragma unroll
                        for (int s = 0; s < STAGES; s += 4) {
                            if (s >= n0) continue;
                            const int4 g = *(const int4 *)(gs + j * ROW + s);
                            const int v0 = row_imax(g.x, last), v1 = row_imax(g.y, last);
                            const int v2 = row_imax(g.z, last), v3 = row_imax(g.w, last);
                            at[s] = v0 < best[s] ? j : at[s];
                            best[s] = row_imin(v0, best[s]);
                            at[s + 1] = v1 < best[s + 1] ? j : at[s + 1];
                            best[s + 1] = row_imin(v1, best[s + 1]);
                            at[s + 2] = v2 < best[s + 2] ? j : at[s + 2];
                            best[s + 2] = row_imin(v2, best[s + 2]);
                            at[s + 3] = v3 < best[s + 3] ? j : at[s + 3];
                            best[s + 3] = row_imin(v3, best[s + 3]);
                        }
                    }
                    if (c0 + t < wd) {
                        const unsigned to = (unsigned)(c0 / LANES) * NS64 + prm_sid(i, 1, r) * 64 + lane;
                        const int base = hidden ? lo_p | PRM_BAND_HIDDEN : lo_p;
#pragma unroll
                        for (int s = 0; s < (STAGES < LANES ? STAGES : LANES - 1); ++s) {
                            if (s >= n0) continue;
                            const unsigned k = to + ((s + 1) * (i + 1) - (s + 1) * (s + 2) / 2) * 64;  // xi = s + 2
                            Wt[k] = best[s];
                            At[k] = (unsigned short)(base + at[s]);
                            atomicMin(Gt + (c0 / LANES) * gsize + (i * (i - 1) / 2 + s + 1) * 64 + lane, best[s]);
                        }
                    }
                }
            }
            if (TEAM) {
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
                __syncthreads();
            }
        }
        if (TEAM) {
            // the best of all waves, of equal ones the fewest replicas
            for (int m = 1; m < team; ++m) {
                if (wib == m) { lds.best[lane] = wbest; lds.best[64 + lane] = rbest; lds.best[128 + lane] = lbest; }
                __syncthreads();
                if (wib == 0) {
                    const int v = lds.best[lane], r = lds.best[64 + lane];
                    if (v < wbest || (v == wbest && r < rbest)) { wbest = v; rbest = r; lbest = lds.best[128 + lane]; }
                }
                __syncthreads();
            }
        }
        // ---- the plans, lane xi - 1 that of xi stages.  (The table was written by other lanes of this workgroup: wait
        // for the stores, then read past the L1 cache, which may hold lines of an earlier candidate.)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        if (have && (!TEAM || wib == 0)) {
            if (bad) {
                if (t == 0) pp_raise(a.status, PP_FAULT_ORDERING);
                if (t < D) a.W_out[c * D + t] = PP_INF64;
                for (int n = t; n < tri; n += LANES) { a.bounds_out[c * tri + n] = 0; a.reps_out[c * tri + n] = 0; }
            } else if (t < D && wbest == INF) {
                // (not with bands that hold a plan, as all do that k_prm_prep finds: its plan is left as it is, because the
                // stores of zeros alone cost 4 us of the 250 that 3001 orderings of 12 GPUs, 75 layers, take)
                a.W_out[c * D + t] = PP_INF64;
            } else if (t < D) {
                const int xi = t + 1;
                a.W_out[c * D + t] = (long long)wbest;
                int *bo = a.bounds_out + c * tri + xi * (xi - 1) / 2, *ro = a.reps_out + c * tri + xi * (xi - 1) / 2;
                int l = L, n = D, r = rbest, cut = lbest, v = wbest;
                bo[xi - 1] = L;
                ro[xi - 1] = r;
                for (int s = xi - 1; s >= 1; --s) {
                    // layers [lp, l) on r replicas as stage s; r' of the stage before: the first one whose value reaches v
                    const int n0 = n - r, nrp = n0 - (s - 1), lp = cut & ~PRM_BAND_HIDDEN;
                    const bool hidden = cut & PRM_BAND_HIDDEN;
                    int rp = n0;
                    if (s > 1) {
                        const int links = __hip_atomic_load(In + (n * 64 + group + n0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const int cell = lp - band[PRM_BAND_LO + n0], place = cell / LANES * (int)NS64 + cell % LANES + group;
                        const int *Ws = Wt + prm_sid(n0, s, 1) * 64 + place;
                        int mf = INF, mb = INF, before = 0, y = 0;
                        bool found = false;
                        // (four values in flight; the last r' is the one if no other is)
                        for (int r0 = 1; !found; r0 += 4) {
                            int four[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                four[u] = __hip_atomic_load(Ws + (row_imin(r0 + u, nrp) - 1) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            if (r0 == 1) {
                                const double den = r < 2 ? 1.0 : (double)r * (double)links, inv = prm_inv(den);
                                y = w.last(w.rec(r, lp, den, inv), w.rec(r, l, den, inv));
                            }
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                if (found) continue;
                                rp = r0 + u;
                                before = four[u];
                                int x = 0;
                                if (!hidden && rp < nrp) {
                                    const int oq = w.o[n0 - rp];
                                    for (int q = n0; q < n; ++q) {
                                        mf = row_imin(mf, w.bw[oq * D + w.o[q]]);
                                        mb = row_imin(mb, w.bw[w.o[q] * D + oq]);
                                    }
                                    x = w.channel(lp, rp * r, mf, mb);
                                }
                                found = rp >= nrp || row_imax(row_imax(before, x), y) == v;
                            }
                        }
                        const int at = prm_sid(n0, s, rp) * 64 + place;
                        v = before;
                        const unsigned *word = (const unsigned *)((uintptr_t)(At + at) & ~(uintptr_t)3);
                        const unsigned two = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        l = lp;
                        cut = (int)((uintptr_t)(At + at) & 2 ? two >> 16 : two & 0xffff);
                    } else {
                        l = lp;
                    }
                    n = n0;
                    r = rp;
                    bo[s - 1] = l;
                    ro[s - 1] = r;
                }
            }
        }
        if (TEAM) __syncthreads();  // (the next candidates' states take these ones' place)
    }
}

// Registers: eight numbers of stages at once take 141; in 128, four waves per SIMD instead of three, a few are spilled.  Teams lose less
// by that than by a round more (7428 orderings of 6 GPUs, 32 layers 96.5 -> 80.6 us, 8150 of 8, 60 layers 145 -> 116; of 8,
// 120 layers, with LDS for two workgroups either way, 207.5 -> 208.3), other launches do not (200 000 of 7, 100 layers 1208 -> 1227).
// With four numbers of stages, which is enough for up to 5 GPUs, 122: 200 000 orderings of 4, 40 layers 279 -> 260 us.
template <int LANES, bool TEAM, int STAGES>
__global__ __launch_bounds__(256, LANES == 8 && (TEAM || STAGES < 8) ? 4 : 3) void k_prm_band(prm_args a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int parts = a.band[PRM_BAND_PARTS];
    if (!parts || a.band[PRM_BAND_LANES] != LANES) return;
    const int D = a.D, L = a.L, L1 = L + 1, tid = threadIdx.x, B = blockDim.x, wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (waves that have room for their states)
    const long long room = (long long)((size_t)a.slots * a.slot_bytes / (parts * prm_band_slot_bytes(D)));
    const long long there = TEAM ? gridDim.x : (long long)gridDim.x * (B >> 6);
    const int waves = (int)(room < there ? room : there);
    double *PA = (double *)smem, *AF = PA + L1, *AB = AF + L1;
    int2 *ut = (int2 *)(AB + L1);
    int4 *rows = (int4 *)(((uintptr_t)(ut + D * L1) + 15) & ~(uintptr_t)15);
    constexpr int EACH = 64 / LANES;
    int *gs = (int *)(rows + (B >> 6) * EACH * prm_band_cells(D, LANES)), *os = gs + (B >> 6) * EACH * prm_band_cells(D, LANES) * prm_band_row(D);
    int *bw = os + B, *band = bw + D * D;
    for (int l = tid; l < L1; l += B) {
        PA[l] = (double)a.pre_out[2 * L1 + l];
        AF[l] = l >= 1 && l < L ? (double)a.actf[l - 1] : 0.0;
        AB[l] = l >= 1 && l < L ? (double)a.actb[l - 1] : 0.0;
    }
    for (int i = tid; i < D * L1; i += B) ut[i] = ((const int2 *)(a.band + PRM_BAND_HDR))[i];
    for (int i = tid; i < D * D; i += B) bw[i] = i / D == i % D ? PP_INF32 : (int)a.bw[i];
    for (int i = tid; i < PRM_BAND_HDR; i += B) band[i] = a.band[i];
    __syncthreads();
    if (tid >= 1 && tid < D) {
        const int lo = band[PRM_BAND_LO + tid], w = band[PRM_BAND_W + tid];
        double f = 0.0, b = 0.0;
        for (int k = lo; k < lo + w && k <= L; ++k) {
            f = AF[k] > f ? AF[k] : f;
            b = AB[k] > b ? AB[k] : b;
        }
        band[PRM_BAND_MOST + tid] = __float_as_int((float)(f + b));
    }
    if (!TEAM) __syncthreads();  // (a team looks there behind the barrier of its first states)
    prm_band_lds lds;
    lds.PA = PA; lds.AF = AF; lds.AB = AB; lds.ut = ut; lds.bw = bw; lds.band = band;
    lds.rows = rows + wib * EACH * prm_band_cells(D, LANES);
    lds.gs = gs + wib * EACH * prm_band_cells(D, LANES) * prm_band_row(D);
    lds.os = os + 64 * wib;
    lds.best = (int *)rows;
    const int wave = TEAM ? blockIdx.x : blockIdx.x * (B >> 6) + wib;
    if (wave < waves) prm_band_run<LANES, TEAM, STAGES>(a, lds, wave, waves, wib, B >> 6);
}

// The launch for LANES lanes per candidate.
template <int LANES>
static void prm_band_launch(const prm_args &a, hipStream_t st) {
    const int wpb = prm_band_waves(a.L, a.D, LANES);
    const size_t lds = prm_band_lds_bytes(a.L, a.D, LANES, wpb);
    const long long room = (long long)((size_t)a.slots * a.slot_bytes / prm_band_slot_bytes(a.D));
    long long sets = (a.N + 64 / LANES - 1) / (64 / LANES);
    // (8000 orderings of 12 GPUs, 2000 waves: 713 us for the call without teams, 727 with; 5040 waves: 434 and 487;
    // 3000 orderings of 16 GPUs, 750 waves: 1438 and 623. )
    const bool team = sets < 1536;
    sets = sets < room ? sets : room;
    sets = sets < 8192 ? sets : 8192;
    const dim3 grid((unsigned)(team ? sets : (sets + wpb - 1) / wpb)), block(64 * wpb);
    constexpr int FEW = LANES == 8 ? 4 : LANES;
    if (a.D <= 5 && team) hipLaunchKernelGGL((k_prm_band<LANES, true, FEW>), grid, block, lds, st, a);
    else if (a.D <= 5) hipLaunchKernelGGL((k_prm_band<LANES, false, FEW>), grid, block, lds, st, a);
    else if (team) hipLaunchKernelGGL((k_prm_band<LANES, true, LANES>), grid, block, lds, st, a);
    else hipLaunchKernelGGL((k_prm_band<LANES, false, LANES>), grid, block, lds, st, a);
}

int pp_launch_prm_band(const prm_args &a, hipStream_t st) {
    hipLaunchKernelGGL(k_prm_prep, dim3(1), dim3(PRM_PREP_THREADS), (size_t)(a.L + 1) * 36, st, a);
    if (a.D <= 8) prm_band_launch<8>(a, st);
    if (a.D > 8 || a.L > prm_band_cells(a.D, 8) + 1) prm_band_launch<16>(a, st);
    return hipGetLastError() == hipSuccess ? PP_OK : PP_ERR_HIP;
}
