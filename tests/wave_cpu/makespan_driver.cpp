// Runs the schedules' kernels that spread a candidate over lanes (their own sources) on the CPU.
// Reads cases from stdin, one per line:
//   run VARIANT S M SEED HI     40 random plans of S stages with times up to HI under the schedule
//                               VARIANT, against Alg. 1's rules written out in 64 bits
//   mixed VARIANT S M SEED HI   the same with 300 plans of times from 0 up: how many were left, how many of
//                               the others differ, and workgroups of the readiness order left in part
//   long VARIANT S M TIME       random plans whose layers' times and transfers are all TIME, under any M: T is the largest of
//                               functions that are linear in M, so that it grows by the longest of its resources' times per
//                               microbatch from where it does so once
//   faulty VARIANT S M N BAD    N plans of which the first BAD have a bad ordering: how many of these have a time, and
//                               how many of the others (a second's work if M is large) have another one than they should
//   launch VARIANT S N          the launches for N candidates (nothing runs): the return value, and how
//                               many candidates they have lanes for
// and prints one line per case.
#include "../../paper_2204_10562_amd/csrc/pp_makespan_split.hip"
#include "../../paper_2204_10562_amd/csrc/pp_makespan_fifo.hip"

#include <string.h>

#include <algorithm>
#include <random>

alignas(16) int rows[16384], lds[16384];  // the kernels' LDS

typedef long long ll;

// Durations: d[j], j = 1..J (block R: the last stage's passes together); lastF, lastB: apart.
static ll reference(int variant, int S, int M, std::vector<ll> d, ll lastF, ll lastB) {
    int R = 2 * S - 1, J = 2 * R - 1;
    if (variant == PP_SCHED_GPIPE) {
        std::vector<ll> busy(R + 2, 0);
        for (int m = 0; m < M; ++m)
            for (int r = 1; r <= R; ++r) busy[r] = std::max(busy[r], r > 1 ? busy[r - 1] : 0) + (r == R ? lastF : d[r]);
        for (int m = 0; m < M; ++m)
            for (int r = R; r >= 1; --r) busy[r] = std::max(busy[r], r < R ? busy[r + 1] : 0) + (r == R ? lastB : d[2 * R - r]);
        return busy[1];
    }
    if (variant == PP_SCHED_ADDITIVE) {
        std::vector<ll> e(2 * S, 0);
        for (int n = 0; n < S; ++n) {
            const int r = 2 * n + 1, in = r - 1, out = 2 * R - in;
            if (n == S - 1) e[S] = d[R] + (n ? d[in] + d[out] : 0);
            else { e[n + 1] = d[r] + (n ? d[in] : 0); e[2 * S - 1 - n] = d[2 * R - r] + (n ? d[out] : 0); }
        }
        d = e; R = S; J = 2 * R - 1;
    }
    if (variant == PP_SCHED_FIFO) {
        // (one item at a time: the earliest start, then the lowest resource; a channel takes the head
        // that was ready first, then the earlier in list order)
        std::vector<int> next(J + 1, 1);
        std::vector<ll> idle(R + 1, 0);
        std::vector<std::vector<ll>> left(J + 1, std::vector<ll>(M + 1, 0));
        for (ll todo = (ll)J * M; todo; --todo) {
            ll first = INT64_MAX;
            int br = 0, bj = 0;
            for (int r = 1; r <= R; ++r) {
                const int ja = r, jb = 2 * R - r, ma = next[ja], mb = jb == ja ? M + 1 : next[jb];
                const bool atA = ma <= M && (ja == 1 || next[ja - 1] > ma), atB = mb <= M && next[jb - 1] > mb;
                const ll ra = atA && ja > 1 ? left[ja - 1][ma] : 0, rb = atB ? left[jb - 1][mb] : 0;
                int j = 0;
                if (r & 1) {
                    if (ma <= M && (mb > M || ma + ja <= mb + jb)) j = atA ? ja : 0;
                    else if (mb <= M) j = atB ? jb : 0;
                } else if (atA && (!atB || ra < rb || (ra == rb && ma + ja <= mb + jb))) j = ja;
                else if (atB) j = jb;
                const ll start = std::max(idle[r], j == ja ? ra : rb);
                if (j && start < first) { first = start; br = r; bj = j; }
            }
            idle[br] = left[bj][next[bj]] = first + d[bj];
            ++next[bj];
        }
        return left[J][M];
    }
    std::vector<ll> fin(J + 2, 0);
    for (int t = 1; t <= M + J - 1; ++t) {
        const std::vector<ll> was = fin;
        for (int pass = 0; pass < 2; ++pass)  // a resource's forward block is served before its backward block
            for (int j = std::max(1, t - M + 1); j <= std::min(J, t); ++j) {
                if ((j > R) != (pass == 1)) continue;
                ll idle = fin[j];
                if (variant != PP_SCHED_DUPLEX || (j & 1)) idle = std::max(idle, fin[2 * R - j]);
                fin[j] = std::max(idle, j > 1 ? was[j - 1] : 0) + d[j];
            }
    }
    return fin[J];
}

struct problem {
    int L, D, S, N;
    std::vector<ll> PF, PB, XF, XB, T;
    std::vector<int> o, e;
    int status = 0;
    mk_args a = {};
    problem(int variant, int S_, int N_, int M, unsigned seed, ll lo, ll hi) : L(S_ + 5), D(S_), S(S_), N(N_) {
        std::mt19937_64 g(seed);
        auto time = [&] { return lo + (ll)(g() % (unsigned long long)(hi - lo + 1)); };
        PF.resize(L + 1);
        PB.resize(L + 1);
        for (int l = 0; l < L; ++l) { PF[l + 1] = PF[l] + time(); PB[l + 1] = PB[l] + time(); }
        XF.resize((size_t)D * D * L);
        XB.resize((size_t)D * D * L);
        for (ll &x : XF) x = time();
        for (ll &x : XB) x = time();
        for (int c = 0; c < N; ++c) {
            std::vector<int> dev(D), cut;
            for (int i = 0; i < D; ++i) dev[i] = i;
            std::shuffle(dev.begin(), dev.end(), g);
            o.insert(o.end(), dev.begin(), dev.begin() + S);
            for (int l = 1; l < L; ++l) cut.push_back(l);
            std::shuffle(cut.begin(), cut.end(), g);
            cut.resize(S - 1);
            std::sort(cut.begin(), cut.end());
            e.insert(e.end(), cut.begin(), cut.end());
            e.push_back(L);
        }
        T.assign(N, -77);
        a.L = L; a.D = D; a.S = S; a.N = N; a.nM = 1;
        for (int &m : a.Ms) m = M;
        a.PF = PF.data(); a.PB = PB.data(); a.XF = XF.data(); a.XB = XB.data();
        a.orderings = o.data(); a.bounds = e.data(); a.T_out = T.data(); a.status = &status;
        a.ord_stride = S; a.bnd_stride = S; a.t_stride = 1;
        a.variant = variant;
    }
    ll want(int c, int M) const {
        const int R = 2 * S - 1, J = 2 * R - 1;
        std::vector<ll> d(J + 2, 0);
        ll lastF = 0, lastB = 0;
        for (int n = 0; n < S; ++n) {
            const int e1 = e[c * S + n], e0 = n ? e[c * S + n - 1] : 0, r = 2 * n + 1;
            const ll F = PF[e1] - PF[e0], B = PB[e1] - PB[e0];
            if (n == S - 1) { d[R] = F + B; lastF = F; lastB = B; }
            else { d[r] = F; d[2 * R - r] = B; }
            if (n) {
                const size_t at = ((size_t)o[c * S + n - 1] * D + o[c * S + n]) * L + e0 - 1;
                d[r - 1] = XF[at];
                d[2 * R - r + 1] = XB[at];
            }
        }
        return reference(a.variant, S, M, d, lastF, lastB);
    }
    // What T grows by per microbatch in a pipeline that is long enough.
    ll slope(int c) const {
        ll most = 0, A = 0, B = 0;
        for (int n = 0; n < S; ++n) {
            const int e1 = e[c * S + n], e0 = n ? e[c * S + n - 1] : 0;
            const size_t at = n ? ((size_t)o[c * S + n - 1] * D + o[c * S + n]) * L + e0 - 1 : 0;
            const ll F = PF[e1] - PF[e0], Bk = PB[e1] - PB[e0], cf = n ? XF[at] : 0, cb = n ? XB[at] : 0;
            A = std::max(A, std::max(F, cf));
            B = std::max(B, std::max(Bk, cb));
            most = std::max(most, a.variant == PP_SCHED_ADDITIVE ? F + Bk + cf + cb
                                  : std::max(F + Bk, a.variant == PP_SCHED_DUPLEX ? std::max(cf, cb) : cf + cb));
        }
        return a.variant == PP_SCHED_GPIPE ? A + B : most;
    }
    int launch() { return a.variant == PP_SCHED_FIFO ? pp_launch_makespan_fifo(a, NULL) : pp_launch_makespan_split(a, NULL); }
};

int main() {
    char what[16];
    while (scanf("%15s", what) == 1) {
        int variant, S;
        ll M, x;
        if (scanf("%d %d %lld", &variant, &S, &M) != 3) return 2;
        if (!strcmp(what, "run")) {
            int seed;
            if (scanf("%d %lld", &seed, &x) != 2) return 2;
            problem p(variant, S, 40, (int)M, seed, variant == PP_SCHED_FIFO ? 1 : 0, x);
            const int rc = p.launch();
            int differ = 0;
            for (int c = 0; c < p.N; ++c) differ += p.T[c] != p.want(c, (int)M);
            printf("%d %d %d\n", rc, p.status, differ);
        } else if (!strcmp(what, "mixed")) {
            int seed;
            if (scanf("%d %lld", &seed, &x) != 2) return 2;
            problem p(variant, S, 300, (int)M, seed, 0, x);
            const int rc = p.launch();
            int left = 0, differ = 0, parts = 0, each = 1;
            while (each < 2 * S - 1) each <<= 1;
            for (int c = 0; c < p.N; ++c) {
                left += p.T[c] == MK_NOT_TAKEN;
                differ += p.T[c] != MK_NOT_TAKEN && p.T[c] != p.want(c, (int)M);
                parts += c % (FIFO_THREADS / each) && (p.T[c] == MK_NOT_TAKEN) != (p.T[c - 1] == MK_NOT_TAKEN);
            }
            printf("%d %d %d %d %d\n", rc, p.status, left, differ, parts);
        } else if (!strcmp(what, "long")) {
            if (scanf("%lld", &x) != 1) return 2;
            problem p(variant, S, 6, (int)M, 1, x, x);
            const int rc = p.launch();
            int differ = 0;
            for (int c = 0; c < p.N; ++c) {
                ll near = 4 * S, slope = p.slope(c);
                while (near < M && p.want(c, (int)near + 1) - p.want(c, (int)near) != slope) near *= 2;
                differ += p.T[c] != (near < M ? p.want(c, (int)near) + (M - near) * slope : p.want(c, (int)M));
            }
            printf("%d %d %d\n", rc, p.status, differ);
        } else if (!strcmp(what, "faulty")) {
            int N, bad;
            if (scanf("%d %d", &N, &bad) != 2) return 2;
            problem p(variant, S, N, (int)M, 5, 1, 9);
            for (int c = 0; c < bad; ++c) p.o[(size_t)c * S + S - 1] = c & 1 ? -1 : S;
            const int rc = p.launch();
            int timed = 0, differ = 0;
            for (int c = 0; c < N; ++c)
                if (c < bad) timed += p.T[c] != PP_INF64;
                else differ += p.T[c] != MK_NOT_TAKEN && p.T[c] != p.want(c, (int)M);
            printf("%d %d %d %d\n", rc, p.status, timed, differ);
        } else {
            problem p(variant, S, 1, 8, 1, 1, 1);
            p.a.N = M;
            p.a.orderings = NULL;
            wave::dry = true;
            wave::launches.clear();
            const int rc = p.launch();
            wave::dry = false;
            // (lanes per candidate: one per resource, rounded up to a power of two, or what the launch says)
            ll lanes = 0;
            for (auto &l : wave::launches) lanes += (ll)l.grid.x * l.block.x;
            int each = 1;
            while (variant == PP_SCHED_FIFO && each < 2 * S - 1) each <<= 1;
            if (variant != PP_SCHED_FIFO) each = (int)wave::launches[0].block.x / 64;
            printf("%d %lld\n", rc, lanes / each);
        }
        fflush(stdout);
    }
    return 0;
}
