// Runs the schedules of plans with replicated stages (k_rep_makespan) on the CPU.  Reads from stdin, one case per line:
//   D L M N SEED HI   N orderings of D GPUs, a random plan of every stage count each, times and sizes up to HI,
//                     against the cost model and Alg. 1's rules written out in 64 bits
// and prints the return value, the status word, how many T differ, and whether the minimum differs.
#include "../../paper_2204_10562_amd/csrc/pp_makespan_rep.hip"

#include <algorithm>
#include <random>

alignas(16) double rep_lds[8192];
alignas(16) int rows[16384];

typedef long long ll;

static ll up(ll x, ll y) { return (x + y - 1) / y; }

int main() {
    int D, L, M, N, seed;
    ll hi;
    while (scanf("%d %d %d %d %d %lld", &D, &L, &M, &N, &seed, &hi) == 6) {
        std::mt19937_64 g(seed);
        auto time = [&](ll lo) { return lo + (ll)(g() % (unsigned long long)(hi - lo + 1)); };
        std::vector<ll> PF(L + 1), PB(L + 1), PA(L + 1), actf(L), actb(L), bw(D * D);
        for (int l = 0; l < L; ++l) {
            PF[l + 1] = PF[l] + time(0); PB[l + 1] = PB[l] + time(0); PA[l + 1] = PA[l] + 50 * time(0);
            actf[l] = 20 * time(0); actb[l] = 20 * time(0);
        }
        for (ll &b : bw) b = 1 + g() % 30;
        const int tri = D * (D + 1) / 2;
        std::vector<int> ord, e((size_t)N * tri, 0), r((size_t)N * tri, 0);
        std::vector<ll> W((size_t)N * D, 7), T((size_t)N * D, -77), want((size_t)N * D);
        for (int c = 0; c < N; ++c) {
            std::vector<int> dev(D);
            for (int i = 0; i < D; ++i) dev[i] = i;
            std::shuffle(dev.begin(), dev.end(), g);
            ord.insert(ord.end(), dev.begin(), dev.end());
            for (int S = 1; S <= D; ++S) {
                auto cuts = [&](int n) {  // S parts of n
                    std::vector<int> at;
                    for (int l = 1; l < n; ++l) at.push_back(l);
                    std::shuffle(at.begin(), at.end(), g);
                    at.resize(S - 1);
                    std::sort(at.begin(), at.end());
                    at.push_back(n);
                    return at;
                };
                ll &out = want[(size_t)c * D + S - 1];
                if (S > L || g() % 16 == 0) { W[(size_t)c * D + S - 1] = out = PP_INF64; continue; }
                const std::vector<int> b = cuts(L), k = cuts(D);
                const size_t at = (size_t)c * tri + S * (S - 1) / 2;
                const int R = 2 * S - 1, J = 2 * R - 1;
                std::vector<ll> d(J + 2, 0), A(S, 0), fin(J + 2, 0);
                for (int s = 0; s < S; ++s) {
                    const int e0 = s ? b[s - 1] : 0, n0 = s ? k[s - 1] : 0, n1 = k[s], q = n1 - n0, before = s ? n0 - (s > 1 ? k[s - 2] : 0) : 0;
                    e[at + s] = b[s];
                    r[at + s] = q;
                    const ll F = up(PF[b[s]] - PF[e0], q), B = up(PB[b[s]] - PB[e0], q);
                    if (s == S - 1) d[R] = F + B;
                    else { d[2 * s + 1] = F; d[2 * R - 2 * s - 1] = B; }
                    ll m = PP_INF64, mf = m, mb = m;
                    for (int v = n0; v < n1; ++v) {
                        for (int u = n0; u < n1; ++u) if (u != v) m = std::min(m, bw[dev[u] * D + dev[v]]);
                        for (int u = n0 - before; u < n0; ++u) {
                            mf = std::min(mf, bw[dev[u] * D + dev[v]]);
                            mb = std::min(mb, bw[dev[v] * D + dev[u]]);
                        }
                    }
                    if (q > 1) A[s] = up(2 * (q - 1) * (PA[b[s]] - PA[e0]), q * m);
                    if (s) {
                        d[2 * s] = up(actf[e0 - 1], (ll)before * q * mf);
                        d[2 * R - 2 * s] = up(actb[e0 - 1], (ll)before * q * mb);
                    }
                }
                for (int t = 1; t <= M + J - 1; ++t) {
                    const std::vector<ll> was = fin;
                    for (int pass = 0; pass < 2; ++pass)
                        for (int j = std::max(1, t - M + 1); j <= std::min(J, t); ++j)
                            if ((j > R) == (pass == 1))
                                fin[j] = std::max(std::max(fin[j], fin[2 * R - j]), j > 1 ? was[j - 1] : 0) + d[j];
                }
                out = fin[J];
                for (int s = 0; s < S; ++s) out = std::max(out, fin[s == S - 1 ? R : 2 * R - 2 * s - 1] + A[s]);
            }
        }
        int status = 0;
        std::vector<tc_pair> part(PP_PARTS);
        std::vector<pp_rep_result> rout(1);
        mk_args a = {};
        a.L = L; a.D = a.S = a.search = D; a.N = N; a.nM = 1;
        for (int &m : a.Ms) m = M;
        a.PF = PF.data(); a.PB = PB.data(); a.PA = PA.data(); a.actf = actf.data(); a.actb = actb.data(); a.bw = bw.data();
        a.orderings = ord.data(); a.bounds = e.data(); a.reps = r.data(); a.W = a.C = W.data(); a.T_out = T.data();
        a.status = &status;
        a.ord_stride = D; a.bnd_stride = tri; a.t_stride = D;
        a.part = part.data(); a.rout = rout.data();
        ll n_part = -1;
        const int rc = mk_launch_replicated(a, NULL, &n_part);
        int differ = 0;
        tc_pair least = {PP_INF64, INT64_MAX}, got = least;
        for (size_t i = 0; i < T.size(); ++i) {
            differ += T[i] != want[i];
            least = tc_min(least, {want[i], (ll)i});
        }
        if (n_part) for (ll i = 0; i < n_part; ++i) got = tc_min(got, part[i]);
        else got = {rout[0].T, rout[0].best_index * D + rout[0].S - 1};
        printf("%d %d %d %d\n", rc, status, differ, (int)(got.T != least.T || got.c != least.c));
        fflush(stdout);
    }
    return 0;
}
