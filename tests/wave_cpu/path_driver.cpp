// Runs the closed form of the schedules (k_makespan_split) on the CPU over plans in memory.  Reads from stdin, one
// case per line:
//   VARIANT S N SEED LO HI SEARCH NM M...   N random plans of S stages (SEARCH: of every stage count up to S)
//                                           with times from LO to HI, under NM microbatch counts, against Alg. 1's rules
//                                           written out in 64 bits, and the minimum over the plans; LO < 0: nothing takes
//                                           any time but two layers, one of them forward and the other backward, and the transfers over
//                                           one cut each way, all of which take HI
// and prints the return value, the status word, how many T differ and how many minima.
#define main makespan_main
#include "makespan_driver.cpp"
#undef main

int main() {
    int variant, S, N, seed, search, nM;
    ll lo, hi;
    while (scanf("%d %d %d %d %lld %lld %d %d", &variant, &S, &N, &seed, &lo, &hi, &search, &nM) == 8) {
        problem p(variant, S, N, 1, seed, lo < 0 ? 0 : lo, lo < 0 ? 0 : hi);
        if (lo < 0) {
            std::mt19937_64 g(seed + 2);
            const int f = g() % p.L, b = g() % p.L, cf = g() % p.L, cb = g() % p.L;
            for (int l = f + 1; l <= p.L; ++l) p.PF[l] = hi;
            for (int l = b + 1; l <= p.L; ++l) p.PB[l] = hi;
            for (int x = 0; x < p.D * p.D; ++x) p.XF[(size_t)x * p.L + cf] = p.XB[(size_t)x * p.L + cb] = hi;
        }
        const int tri = search ? S * (S + 1) / 2 : S, xs = search ? S : 1;
        for (int q = 0; q < nM; ++q) if (scanf("%d", &p.a.Ms[q]) != 1) return 2;
        std::vector<int> e;
        std::mt19937_64 g(seed + 1);
        for (int c = 0; c < N; ++c)
            for (int xi = search ? 1 : S; xi <= S; ++xi) {
                std::vector<int> cut;
                for (int l = 1; l < p.L; ++l) cut.push_back(l);
                std::shuffle(cut.begin(), cut.end(), g);
                cut.resize(xi - 1);
                std::sort(cut.begin(), cut.end());
                e.insert(e.end(), cut.begin(), cut.end());
                e.push_back(p.L);
            }
        std::vector<ll> T((size_t)nM * N * xs, -77), C((size_t)N * xs, 5);
        std::vector<tc_pair> part(PP_PARTS * PP_MAX_M_LIST);
        std::vector<pp_result> out(PP_MAX_M_LIST);
        p.a.nM = nM;
        p.a.search = search ? S : 0;
        p.a.bounds = e.data();
        p.a.bnd_stride = tri;
        p.a.t_stride = xs;
        p.a.T_out = T.data();
        p.a.C = C.data();
        p.a.part = part.data();
        p.a.out = out.data();
        long long n_part = -1;
        const int rc = pp_launch_makespan_split(p.a, NULL, &n_part);
        int differ = 0, minima = 0;
        for (int q = 0; q < nM; ++q) {
            tc_pair least = {PP_INF64, INT64_MAX}, got = least;
            for (int c = 0; c < N; ++c)
                for (int x = 0; x < xs; ++x) {
                    problem one = p;
                    one.S = search ? x + 1 : S;
                    one.o.assign(p.o.begin() + (size_t)c * S, p.o.begin() + (size_t)c * S + one.S);
                    const size_t at = (size_t)c * tri + (search ? x * (x + 1) / 2 : 0);
                    one.e.assign(e.begin() + at, e.begin() + at + one.S);
                    const ll t = one.want(0, p.a.Ms[q]), at_T = ((ll)q * N + c) * xs + x;
                    differ += T[at_T] != t;
                    least = tc_min(least, {t, (ll)c * xs + x});
                }
            if (n_part) for (ll i = 0; i < n_part; ++i) got = tc_min(got, part[q * n_part + i]);
            else got = {out[q].T, search ? out[q].best_index * S + out[q].S - 1 : out[q].best_index};
            minima += got.T != least.T || got.c != least.c;
        }
        printf("%d %d %d %d\n", rc, p.status, differ, minima);
        fflush(stdout);
    }
    return 0;
}
