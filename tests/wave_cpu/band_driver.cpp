// Runs the partition from a few cells per row (pp_dp_band.h, its own source) on the CPU: the block that finds the
// bands, the words of the links, and the pass over the candidates.  Reads cases from stdin, one per line:
//   L D S N SEED KIND STAGES WORDS
// KIND: what the layer and transfer times look like (below); STAGES: plans of every number of stages; WORDS: whether
// the words of the links are there.  Prints, per case, the return value, the status, how many results of the
// candidates that ended differ from the recursion over all splits, how many ended, and how many candidates with a
// bad ordering were reported; with an argument also the work counters: pairs, rows, and those of them in bands and
// of the channel-free program.  The list counts as one that is long enough for the recursion, with the argument
// "short" as one that is not.  With the argument "layout" the cases are L D S N, and what is printed is whether
// there is room for what k_band_free leaves, and whether a part of it lies where something else is at that time.
// With the argument "free" (STAGES 0, WORDS 1) the candidates with the channel-free plan are also scheduled where they are
// found, and printed are how many of these there are, how many of their T differ from Alg. 1's rules for the plan of the recursion, how many
// minima of 64 are wrong, and how many candidates have both been scheduled and left something (bounds, or a bit for the DP kernel).
#define main makespan_main
#include "makespan_driver.cpp"
#undef main

#include "../../paper_2204_10562_amd/csrc/pp_dp_band_table.h"
#include "../../paper_2204_10562_amd/csrc/pp_dp_band.hip"

alignas(16) unsigned char smem[64 * 1024];  // the kernels' LDS
alignas(16) long long dyn[8 * 1024];

static void k_band_table(band_table_args a) { band_table(a, (unsigned char *)dyn); }

int main(int argc, char **argv) {
    const bool shorter = argc > 1 && !strcmp(argv[1], "short"), frees = argc > 1 && !strcmp(argv[1], "free");
    int L, D, S, N, seed, kind, stages, words;
    if (argc > 1 && !strcmp(argv[1], "layout")) {
        while (scanf("%d %d %d %d", &L, &D, &S, &N) == 4) {
            const pp_ws_layout w = pp_layout(L, D, S, N);
            const size_t groups = (N + 63) / 64, lower = w.sh_rows ? (size_t)N * 4 : groups * 8;  // the list, or the bits
            const size_t times = w.fx + (size_t)D * D * S * 8;
            bool clash = w.fbits < w.left + lower || w.fleast < w.fbits + groups * 8 || w.fleast + groups * 8 * PP_FREE_COUNTS > w.part;
            clash |= w.sh_rows ? w.fx != w.sh_rows || times > w.total : w.fx != w.arg || times > w.band;
            clash |= (w.fx | w.fbits | w.fleast) & 7;
            printf("%d %d\n", w.fx != 0, w.fx && clash);
        }
        return 0;
    }
    while (scanf("%d %d %d %d %d %d %d %d", &L, &D, &S, &N, &seed, &kind, &stages, &words) == 8) {
        std::mt19937_64 g(seed);
        auto upto = [&](ll n) { return (ll)(g() % (unsigned long long)(n + 1)); };
        std::vector<ll> PF(L + 1), PB(L + 1, 0), P(L + 1);
        std::vector<ll> XF((size_t)D * D * L), XB((size_t)D * D * L, 0);
        for (int l = 0; l < L; ++l) {
            ll t = 50 + upto(950);
            if (kind == 1 && upto(2) == 0) t = 0;                  // a third of the layers of length zero
            if (kind == 2) t = 1 + upto(2);                        // ties everywhere
            if (kind == 3 && l == L / 2) t = 40000;                // one layer outweighs the others
            if (kind == 4) t = 100;                                // equal layers
            PF[l + 1] = P[l + 1] = P[l] + t;
        }
        const ll top = P[L] / S + 1;
        for (int i = 0; i < D * D; ++i)
            for (int k = 0; k < L; ++k) {
                ll x = upto(top / 2);
                if (kind == 5) x = upto(top + top / 2);            // links that bind now and then
                if (kind == 6) x = upto(4 * top);                  // and nearly everywhere
                if (kind == 7) x = top / 2 + upto(top);
                XF[(size_t)i * L + k] = x;
            }
        std::vector<int> ord((size_t)N * S);
        for (int c = 0; c < N; ++c) {
            std::vector<int> dev(D);
            for (int i = 0; i < D; ++i) dev[i] = i;
            std::shuffle(dev.begin(), dev.end(), g);
            std::copy(dev.begin(), dev.begin() + S, ord.begin() + (size_t)c * S);
        }
        // (half of some layers' times, and of transfers, the other way)
        for (int l = 0; frees && l < L; ++l) PB[l + 1] = PB[l] + (P[l + 1] - P[l]) / (2 + l % 3);
        for (int l = 0; l <= L; ++l) PF[l] = P[l] - PB[l];
        std::vector<ll> X = XF;
        for (size_t i = 0; frees && i < XF.size(); ++i) { XB[i] = X[i] / (2 + i % 3); XF[i] = X[i] - XB[i]; }
        const int bad = N / 3;
        if (kind == 0) ord[(size_t)bad * S + S - 1] = ord[(size_t)bad * S];
        static pp_ws_header hdr;
        memset(&hdr, 0, sizeof hdr);
        ll vmax = P[L];
        for (ll x : X) vmax = std::max(vmax, x);
        hdr.pmax[3] = (unsigned long long)vmax;
        std::vector<int> p32(L + 17, (int)P[L]), x32((size_t)D * D * L + 129, 0x55555555);
        for (int l = 0; l <= L; ++l) p32[l] = (int)P[l];
        for (size_t i = 0; i < (size_t)D * D * L; ++i) x32[i] = i % L ? (int)X[i - 1] : 0;
        const int tri = stages ? S * (S + 1) / 2 : S, nc = stages ? S : 1;
        std::vector<int> table((size_t)S * 700, 0x7abcdef);
        std::vector<unsigned long long> links(band_link_words(D, S, stages)), left((N + 63) / 64);
        std::vector<ll> C((size_t)N * nc, -7);
        std::vector<int> bounds((size_t)N * tri + 4, -7);
        int status = 0;
        band_table_args p = {};
        p.L = L; p.D = D; p.S = S; p.K = pp_index_bits(L);
        p.PF = PF.data(); p.PB = PB.data(); p.XF = XF.data(); p.XB = XB.data();
        p.table = table.data(); p.stages = stages; p.cells = shorter ? 0 : 2;
        p.fit_limit = (1ull << (31 - p.K)) - 1;
        const size_t need = band_table_lds(L, S, stages, p.waves);
        if (need > sizeof dyn) return 1;
        memset(dyn, seed & 255, sizeof dyn);
        memset(smem, seed & 255, sizeof smem);
        wave::launch(k_band_table, dim3(1), dim3(256), need, p);
        dp_args a = {};
        a.L = L; a.D = D; a.S = S; a.K = p.K; a.N = N;
        a.validate = 1;
        a.fit_limit = p.fit_limit;
        a.hdr = &hdr; a.p32 = p32.data(); a.x32 = x32.data(); a.ord = ord.data();
        a.stages = stages; a.C_out = C.data(); a.bounds_out = bounds.data(); a.status = &status;
        a.band = table.data();
        a.band_all = shorter ? N + 1 : N;
        a.PF = PF.data(); a.PB = PB.data(); a.XF = XF.data(); a.XB = XB.data();
        const int groups = (N + 63) / 64, nM = 1 + seed % PP_FREE_COUNTS, Ms[] = {2 + seed % 5, 19, 5, 40};
        std::vector<int2> fx((size_t)D * D * S);
        std::vector<unsigned long long> bits(groups, 0);
        std::vector<ll> T((size_t)nM * N, -7), least((size_t)nM * groups, -7);
        if (frees) {
            a.fx = fx.data(); a.fbits = bits.data(); a.fT = T.data(); a.fleast = least.data();
            a.f_nM = nM;
            for (int q = 0; q < PP_FREE_COUNTS; ++q) a.f_Ms[q] = q < nM ? Ms[q] : 1;
        }
        const int rc = pp_launch_dp_band_alone(a, words ? links.data() : NULL, left.data(), NULL);
        int differ = 0, ended = 0, reported = 0, scheduled = 0, times = 0, minima = 0, both = 0;
        const int *plan = table.data() + band_plan_at(S, S);
        std::vector<ll> lowest((size_t)nM * groups, -1);
        for (int c = 0; c < N; ++c) {
            // (without bands the pass does nothing, and the kernel behind it looks at nothing it has left)
            if (table[band_top_at(S, 0, S)] < 0 || (left[c >> 6] >> (c & 63) & 1)) continue;
            if (kind == 0 && c == bad) {
                reported += C[(size_t)c * nc] == INT64_MAX;
                continue;
            }
            ++ended;
            std::vector<std::vector<ll>> W(S, std::vector<ll>(L + 1));
            std::vector<std::vector<int>> A(S, std::vector<int>(L + 1));
            W[0] = P;
            for (int n = 1; n < S; ++n)
                for (int l = 0; l <= L; ++l) {
                    W[n][l] = INT64_MAX;
                    for (int k = n; k < l; ++k) {
                        const ll x = x32[((size_t)ord[(size_t)c * S + n - 1] * D + ord[(size_t)c * S + n]) * L + k];
                        const ll v = std::max(std::max(W[n - 1][k], x), P[l] - P[k]);
                        if (v < W[n][l]) { W[n][l] = v; A[n][l] = k; }
                    }
                }
            if (hdr.free_valid && (bits[c >> 6] >> (c & 63) & 1)) {
                ++scheduled;
                both += left[c >> 6] >> (c & 63) & 1;
                for (int n = 0; n < S; ++n) both += bounds[(size_t)c * S + n] != -7;
                differ += C[c] != W[S - 1][L];
                for (int n = S - 1, e = L; n >= 0; --n) {
                    differ += plan[n] != e;
                    e = A[n][e];
                }
                const int R = 2 * S - 1;
                std::vector<ll> d(2 * R + 1, 0);
                for (int n = 0; n < S; ++n) {
                    const int e0 = n ? plan[n - 1] : 0, r = 2 * n + 1;
                    const ll F = PF[plan[n]] - PF[e0], B = PB[plan[n]] - PB[e0];
                    d[r] = n == S - 1 ? F + B : F;
                    if (n < S - 1) d[2 * R - r] = B;
                    if (!n) continue;
                    const size_t at = ((size_t)ord[(size_t)c * S + n - 1] * D + ord[(size_t)c * S + n]) * L + e0 - 1;
                    d[r - 1] = XF[at];
                    d[2 * R - r + 1] = XB[at];
                }
                for (int q = 0; q < nM; ++q) {
                    const ll t = reference(PP_SCHED_PE, S, Ms[q], d, 0, 0), v = t << 6 | (c & 63);
                    times += T[(size_t)q * N + c] != t;
                    ll &l = lowest[(size_t)q * groups + (c >> 6)];
                    if (l < 0 || v < l) l = v;
                }
                continue;
            }
            for (int xi = stages ? 1 : S; xi <= S; ++xi) {
                differ += C[(size_t)c * nc + (stages ? xi - 1 : 0)] != W[xi - 1][L];
                const int *b = &bounds[(size_t)c * tri + (stages ? xi * (xi - 1) / 2 : 0)];
                for (int n = xi - 1, e = L; n >= 0; --n) {
                    differ += b[n] != e;
                    e = A[n][e];
                }
            }
        }
        for (int i = 0; hdr.free_valid && i < nM * groups; ++i) minima += least[i] != lowest[i];
        printf("%d %d %d %d %d", rc, status, differ, ended, reported);
        if (frees) {
            printf(" %d %d %d %d\n", scheduled, times, minima, both);
            fflush(stdout);
            continue;
        }
        ll work[5] = {};
        for (auto &w : hdr.work) {
            work[0] += w.pairs; work[1] += w.rows; work[2] += w.band_pairs; work[3] += w.band_rows; work[4] += w.free_rows;
        }
        for (ll w : work) if (argc > 1) printf(" %lld", w);
        printf("\n");
        fflush(stdout);
    }
    return 0;
}
