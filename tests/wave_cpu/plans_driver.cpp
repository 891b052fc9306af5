// Runs the schedules of the planner's own plans (k_makespan_plans) on the CPU over plans in memory.  Reads from stdin, one
// case per line:
//   S N SEED HI SEARCH FREE NM M...   N random plans of S stages (SEARCH: of every stage count up to S) with times up to HI
//                                     under NM microbatch counts, against Alg. 1's rules written out in 64 bits.  Some
//                                     orderings are bad, and some plans have a bound that is none.  FREE: about half of
//                                     the candidates, and whole groups of 64, have been scheduled already (their bounds
//                                     are anything)
// and prints the return value, the status word, how many T differ, how many winners, and how many plans were torn.
#define main makespan_main
#include "makespan_driver.cpp"
#undef main

#include <sys/mman.h>

// The values, and no page behind them that can be read.
static ll *guarded(const std::vector<ll> &v) {
    const size_t page = 4096, bytes = (v.size() * 8 + page - 1) / page * page, gap = 16 << 20;
    char *p = (char *)mmap(NULL, bytes + gap, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED || mprotect(p, bytes, PROT_READ | PROT_WRITE)) abort();
    ll *at = (ll *)(p + bytes - v.size() * 8);
    std::copy(v.begin(), v.end(), at);
    return at;
}

int main() {
    int S, N, seed, search, free_some, nM;
    ll hi;
    while (scanf("%d %d %d %lld %d %d %d", &S, &N, &seed, &hi, &search, &free_some, &nM) == 7) {
        problem p(PP_SCHED_PE, S, N, 1, seed, 0, hi);
        const int tri = search ? S * (S + 1) / 2 : S, xs = search ? S : 1;
        for (int q = 0; q < nM; ++q) if (scanf("%d", &p.a.Ms[q]) != 1) return 2;
        std::mt19937_64 g(seed + 1);
        std::vector<int> e, plan(64, 0);
        std::vector<bool> torn((size_t)N * xs, false), bad(N, false);
        std::vector<ll> C((size_t)N * xs), T((size_t)nM * N * xs, -77), want(T.size());
        const int groups = (N + 63) / 64;
        std::vector<unsigned long long> bits(groups, 0);
        for (int c = 0; free_some && c < N; ++c)
            if ((c / 64) % 3 == 1 || g() % 2) bits[c / 64] |= 1ull << (c % 64);
        for (int n = 0; n < S; ++n) plan[n] = n < S - 1 ? n + 1 : p.L;
        for (int c = 0; c < N; ++c) {
            const bool done = bits[c / 64] >> (c % 64) & 1;
            bad[c] = !done && S > 1 && g() % 16 == 0;
            for (int xi = search ? 1 : S; xi <= S; ++xi) {
                const size_t k = (size_t)c * xs + (search ? xi - 1 : 0);
                std::vector<int> cut;
                for (int l = 1; l < p.L; ++l) cut.push_back(l);
                std::shuffle(cut.begin(), cut.end(), g);
                cut.resize(xi - 1);
                std::sort(cut.begin(), cut.end());
                cut.push_back(p.L);
                problem one = p;
                one.S = xi;
                one.o.assign(p.o.begin() + (size_t)c * S, p.o.begin() + (size_t)c * S + xi);
                one.e = cut;
                C[k] = 2 * (p.L + 1) * hi;  // (no time is longer)
                for (int q = 0; q < nM; ++q) want[((size_t)q * N + c) * xs + (search ? xi - 1 : 0)] = one.want(0, p.a.Ms[q]);
                const int none[] = {0, -1, p.L + 1, 65535, 1 << 30};
                torn[k] = !done && !bad[c] && hi > 3 && g() % 16 == 0;
                if (torn[k]) cut[g() % xi] = none[g() % 5];
                if (done) for (int &x : cut) x = (int)g();
                e.insert(e.end(), cut.begin(), cut.end());
                if (bad[c]) C[k] = PP_INF64;
                if (bad[c] || torn[k])
                    for (int q = 0; q < nM; ++q) want[((size_t)q * N + c) * xs + (search ? xi - 1 : 0)] = PP_INF64;
            }
            if (bad[c]) p.o[(size_t)c * S] = c & 1 ? p.D : -1;  // (in the plans of every stage count)
        }
        // what k_band_free leaves: T, and the least of 64 with its place
        std::vector<ll> least((size_t)nM * groups, -1);
        for (int c = 0; c < N; ++c)
            if (bits[c / 64] >> (c % 64) & 1)
                for (int q = 0; q < nM; ++q) {
                    const ll t = want[(size_t)q * N + c], v = t << 6 | (c % 64);
                    T[(size_t)q * N + c] = t;
                    ll &l = least[(size_t)q * groups + c / 64];
                    if (l < 0 || t < l >> 6) l = v;
                }
        static pp_ws_header hdr;
        hdr.free_valid = free_some;
        std::vector<tc_pair> part(PP_PARTS * PP_MAX_M_LIST);
        std::vector<pp_result> out(PP_MAX_M_LIST);
        p.a.XF = guarded(p.XF);
        p.a.XB = guarded(p.XB);
        p.a.nM = nM; p.a.search = search ? S : 0;
        p.a.orderings = p.o.data(); p.a.bounds = e.data(); p.a.bnd_stride = tri; p.a.t_stride = xs;
        p.a.T_out = T.data(); p.a.C = C.data(); p.a.part = part.data(); p.a.out = out.data(); p.a.hdr = &hdr;
        if (free_some) { p.a.free_bits = bits.data(); p.a.free_least = least.data(); p.a.free_plan = plan.data(); }
        long long n_part = -1;
        const int rc = pp_launch_makespan_split(p.a, NULL, &n_part);
        int differ = 0, winners = 0, tears = 0;
        for (size_t i = 0; i < T.size(); ++i) differ += T[i] != want[i];
        for (int q = 0; q < nM; ++q) {
            tc_pair first = {PP_INF64, INT64_MAX}, got = first;
            for (ll i = 0; i < (ll)N * xs; ++i) first = tc_min(first, {want[(size_t)q * N * xs + i], i});
            if (n_part) for (ll i = 0; i < n_part; ++i) got = tc_min(got, part[q * n_part + i]);
            else if (first.T == PP_INF64) got = {out[q].T, out[q].best_index == -1 ? INT64_MAX : 0};
            else got = {out[q].T, search ? out[q].best_index * S + out[q].S - 1 : out[q].best_index};
            winners += got.T != first.T || (first.T != PP_INF64 && got.c != first.c);
        }
        for (size_t k = 0; k < torn.size(); ++k) tears += torn[k];
        printf("%d %d %d %d %d\n", rc, p.status, differ, winners, tears);
        fflush(stdout);
    }
    return 0;
}
