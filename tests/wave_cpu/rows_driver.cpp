// Runs the partition DP's kernels that search for a cell's split (their own sources) on the CPU: the row
// kernel for L <= 128, the one for longer rows beyond.  Reads cases from stdin, one per line:
//   L D S N SEED KIND STAGES FILL
// KIND: what the layer and transfer times look like (see problem below); STAGES: plans of every number
// of stages; FILL: the byte the LDS is filled with before the launch.  Prints, per case, the return value,
// the status, how many results differ from the recursion over all splits, the steps the kernel counted, and
// a number that depends on all votes its waves took.  With an argument (L <= 128) some candidates are finished
// before the kernel runs, as a launch of bands leaves them: in runs of 64, nine in ten of a run left, a few or none.
// Theirs are to stay as they are: a result of theirs that the kernel writes counts as a difference.  With the argument
// "bad" none is finished, and some orderings name a device twice, which are to have no plan: of a wave's candidates 70 after
// every 32, or one in four.
#include "../../paper_2204_10562_amd/csrc/pp_dp_rows.hip"
#include "../../paper_2204_10562_amd/csrc/pp_dp_big.hip"

#include <string.h>

#include <algorithm>
#include <random>

alignas(16) unsigned char smem[64 * 1024];  // the kernel's LDS

typedef long long ll;

int main(int argc, char **argv) {
    const bool bad = argc > 1 && !strcmp(argv[1], "bad");
    int L, D, S, N, seed, kind, stages, fill;
    while (scanf("%d %d %d %d %d %d %d %d", &L, &D, &S, &N, &seed, &kind, &stages, &fill) == 8) {
        std::mt19937_64 g(seed);
        auto upto = [&](ll n) { return (ll)(g() % (unsigned long long)(n + 1)); };
        std::vector<ll> P(L + 1);
        std::vector<int> X((size_t)D * D * L);
        for (int l = 0; l < L; ++l) {
            ll t = 50 + upto(950);
            if (kind == 1 && l == L / 3) t = 0;                    // one layer of length zero
            if ((kind == 2 || kind == 9) && upto(1)) t = 0;        // half of them
            if (kind == 3 && l == L - 1) t = 2 * P[l];             // the last layer outweighs the others
            if (kind == 4) t = l < 3 * L / 4 ? 1 : 400;            // most layers in little time
            if (kind == 7) t = 0;
            P[l + 1] = P[l] + t;
        }
        const ll top = P[L] / S + 1;
        for (int i = 0; i < D * D; ++i) {
            const ll slow = kind == 5 || kind == 6 ? 1 + upto(8) : 1;
            for (int k = 0; k < L; ++k) {
                ll x = upto(top / 8 + 1);
                if (kind == 5) x = slow * top * (L - k) / L;       // every cut cheaper than the one before
                if (kind == 6) x = upto(slow * top);               // links bind everywhere, in no order
                if (kind <= 2 && k % 5 == 0) x = 3 * top;          // a few cuts that cost more than a stage
                if (kind >= 8) x = k % 47 == 5 ? 3 * top : 1;          // one cut in 47 of those
                X[(size_t)i * L + k] = (int)x;                     // [k]: the cut between layers k - 1 and k
            }
        }
        std::vector<int> ord((size_t)N * S);
        for (int c = 0; c < N; ++c) {
            std::vector<int> dev(D);
            for (int i = 0; i < D; ++i) dev[i] = i;
            if (c && upto(2)) {                                    // (neighbours share devices)
                dev.assign(ord.begin() + (size_t)(c - 1) * S, ord.begin() + (size_t)c * S);
                for (int i = 0; i < D; ++i)
                    if (std::find(dev.begin(), dev.end(), i) == dev.end()) dev.push_back(i);
                std::shuffle(dev.begin() + upto(S - 1), dev.end(), g);
            } else {
                std::shuffle(dev.begin(), dev.end(), g);
            }
            std::copy(dev.begin(), dev.begin() + S, ord.begin() + (size_t)c * S);
            // (one in two as the one before its neighbour: rows to share with what a wave has done before)
            if (argc > 1 && c >= 2 && upto(1)) std::copy_n(ord.begin() + (size_t)(c - 2) * S, S, ord.begin() + (size_t)c * S);
        }
        std::vector<char> twice(N, 0);
        for (int c = 0; bad && c < N; ++c)
            if (seed & 1 ? !upto(3) : c % ((N + 2) / 3) % 102 >= 32) {
                twice[c] = 1;
                ord[(size_t)c * S + S - 1] = ord[(size_t)c * S];
            }
        static pp_ws_header hdr;
        memset(&hdr, 0, sizeof hdr);
        ll vmax = P[L];
        for (int x : X) vmax = std::max(vmax, (ll)x);
        hdr.pmax[3] = (unsigned long long)vmax;
        std::vector<int> p32(L + 17, (int)P[L]), x32 = X;
        for (int l = 0; l <= L; ++l) p32[l] = (int)P[l];
        x32.resize(X.size() + 129, 0x55555555);                    // (what follows the table in the workspace)
        const int tri = stages ? S * (S + 1) / 2 : S, nc = stages ? S : 1;
        std::vector<ll> C((size_t)N * nc, -7);
        std::vector<int> bounds((size_t)N * tri, -7);
        int status = 0;
        dp_args a = {};
        a.L = L; a.D = D; a.S = S; a.K = pp_index_bits(L); a.N = N;
        a.validate = 1;
        a.fit_limit = (1ull << (31 - a.K)) - 1;
        a.hdr = &hdr; a.p32 = p32.data(); a.x32 = x32.data(); a.ord = ord.data();
        a.stages = stages; a.C_out = C.data(); a.bounds_out = bounds.data(); a.status = &status;
        a.nblocks = 3;
        std::vector<unsigned short> arg((size_t)3 * S * (L + 128));
        a.arg = arg.data();
        memset(smem, fill, sizeof smem);
        wave::votes = 1;
        std::vector<unsigned long long> left((N + 63) / 64, ~0ull);
        std::vector<int> band((size_t)S * 700, 0);  // (there are bands)
        int rc;
        if (L > PP_TILE_MAX_L) {
            rc = pp_launch_dp_big(a, 3, 256, NULL, NULL);          // three waves share the list
        } else {
            dp_rows_args t = {};
            t.L = L; t.D = D; t.S = S; t.K = a.K; t.N = N;
            t.validate = 1;
            t.chunk = (N + 2) / 3;
            if (argc > 1 && !bad) {
                std::fill(left.begin(), left.end(), 0);
                for (int c = 0; c < N; ++c) {
                    const int often = (int[]){9, 1, 0, 10, 5}[c / 64 % 5];
                    if (upto(9) < often) left[c >> 6] |= 1ull << (c & 63);
                }
                a.band = band.data();
                a.left = left.data();
            }
            t.g = a;
            const dpr_shape sh = pp_dp_rows_shape(L, D, S, stages);
            rc = pp_launch_dp_rows(t, (3 + sh.wpb - 1) / sh.wpb, sh, NULL);
        }
        int differ = 0;
        for (int c = 0; c < N; ++c) {
            if (!(left[c >> 6] >> (c & 63) & 1)) {
                for (int i = 0; i < nc; ++i) differ += C[(size_t)c * nc + i] != -7;
                for (int i = 0; i < tri; ++i) differ += bounds[(size_t)c * tri + i] != -7;
                continue;
            }
            if (twice[c]) {
                for (int i = 0; i < nc; ++i) differ += C[(size_t)c * nc + i] != INT64_MAX;
                for (int i = 0; i < tri; ++i) differ += bounds[(size_t)c * tri + i] != 0;
                continue;
            }
            std::vector<std::vector<ll>> W(S, std::vector<ll>(L + 1));
            std::vector<std::vector<int>> A(S, std::vector<int>(L + 1));
            W[0] = P;
            for (int n = 1; n < S; ++n)
                for (int l = 0; l <= L; ++l) {
                    W[n][l] = INT64_MAX;
                    for (int k = n; k < l; ++k) {
                        const ll x = X[((size_t)ord[(size_t)c * S + n - 1] * D + ord[(size_t)c * S + n]) * L + k];
                        const ll v = std::max(std::max(W[n - 1][k], x), P[l] - P[k]);
                        if (v < W[n][l]) { W[n][l] = v; A[n][l] = k; }
                    }
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
        ll pairs = 0;
        for (auto &r : hdr.work) pairs += (ll)r.pairs;
        printf("%d %d %d %lld %llu\n", rc, status, differ, pairs, wave::votes);
        fflush(stdout);
    }
    return 0;
}
