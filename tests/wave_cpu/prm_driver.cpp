// Runs the replicated planner from the bands (pp_prm_band.hip, its own source) on the CPU: the workgroup that finds the
// bands, then the kernel that plans every candidate from them.  Reads problems from stdin as numbers:
//   L D N M TEAM fwd[L] bwd[L] actf[L] actb[L] alpha[L] bw[D*D] ord[N*D]
// TEAM: whether the waves of a workgroup share candidates.  Prints, per problem, the status, the parts of a band (0: the
// bands are not used), the lanes per candidate, the widest band, whether times for it were tried, and, where bands are
// used, W, bounds and replicas of every candidate.  With L = 0 the last number of layers up to which there can be bands
// of D devices, up to which a workgroup has four waves (8 and 16 lanes a candidate), and up to which three of those with 16
// lanes share the 160 KB of a compute unit.
#include <hip/hip_runtime.h>

#undef __shared__
#define __shared__ thread_local  // (the fibers of a workgroup are one thread)

#include "../../paper_2204_10562_amd/csrc/pp_prm_band.hip"

#include <algorithm>

thread_local alignas(16) unsigned char smem[64 * 1024];  // the kernels' LDS

typedef long long ll;

template <int LANES>
static void plan(const prm_args &a, bool team) {
    const int wpb = prm_band_waves(a.L, a.D, LANES);
    const size_t lds = prm_band_lds_bytes(a.L, a.D, LANES, wpb);
    if (lds > sizeof smem) abort();
    constexpr int FEW = LANES == 8 ? 4 : LANES;
    if (a.D <= 5 && team) wave::launch(k_prm_band<LANES, true, FEW>, dim3(2), dim3(64 * wpb), lds, a);
    else if (a.D <= 5) wave::launch(k_prm_band<LANES, false, FEW>, dim3(2), dim3(64 * wpb), lds, a);
    else if (team) wave::launch(k_prm_band<LANES, true, LANES>, dim3(2), dim3(64 * wpb), lds, a);
    else wave::launch(k_prm_band<LANES, false, LANES>, dim3(2), dim3(64 * wpb), lds, a);
}

int main() {
    int L, D, N, M, team;
    while (scanf("%d %d %d %d %d", &L, &D, &N, &M, &team) == 5) {
        if (L == 0) {
            int last = 0, four8 = 0, four16 = 0, three = 0;
            for (int l = D; l <= 1024; ++l) {
                const int w8 = prm_band_waves(l, D, 8), w16 = prm_band_waves(l, D, 16);
                if (w8 && w16) last = l;
                if (w8 == 4) four8 = l;
                if (w16 == 4) four16 = l;
                if (w8 && w16 && 3 * prm_band_lds_bytes(l, D, 16, w16) <= 160 * 1024) three = l;
            }
            printf("%d %d %d %d\n", last, four8, four16, three);
            continue;
        }
        auto read = [&](size_t n) {
            std::vector<ll> v(n);
            for (ll &x : v) if (scanf("%lld", &x) != 1) exit(1);
            return v;
        };
        const std::vector<ll> fwd = read(L), bwd = read(L), actf = read(L), actb = read(L), alpha = read(L), bw = read((size_t)D * D);
        const std::vector<ll> o = read((size_t)N * D);
        const std::vector<int> ord(o.begin(), o.end());
        const int tri = D * (D + 1) / 2;
        std::vector<ll> W((size_t)N * D, -7), pre(3 * (size_t)(L + 1));
        std::vector<int> bounds((size_t)N * tri, -7), reps((size_t)N * tri, -7), band(prm_band_bytes(L, D) / 4, 0x55555555);
        prm_args a = {};
        a.L = L; a.D = D; a.M = M; a.N = N;
        a.fwd = fwd.data(); a.bwd = bwd.data(); a.actf = actf.data(); a.actb = actb.data();
        a.alpha = alpha.data(); a.bw = bw.data(); a.ord = ord.data();
        a.slots = 3;  // (fewer than the waves: some of them plan several sets of candidates)
        a.slot_bytes = 2 * prm_band_slot_bytes(D);
        std::vector<char> scratch(a.slots * a.slot_bytes + 64, 0x55);
        a.scratch = scratch.data();
        a.W_out = W.data(); a.bounds_out = bounds.data(); a.reps_out = reps.data();
        a.pre_out = pre.data();
        a.band = band.data();
        int status = 0;
        a.status = &status;
        if (!prm_band_wanted(a)) return 1;
        wave::launch(k_prm_prep, dim3(1), dim3(PRM_PREP_THREADS), (size_t)(L + 1) * 36, a);
        const int parts = band[PRM_BAND_PARTS], lanes = parts ? band[PRM_BAND_LANES] : 0;
        int widest = 0;
        for (int i = 1; parts && i < D; ++i) widest = std::max(widest, band[PRM_BAND_W + i]);
        plan<8>(a, team);  // (does nothing where the other has the launch)
        plan<16>(a, team);
        for (int i = 0; i < 64; ++i) if (scratch[a.slots * a.slot_bytes + i] != 0x55) return 1;
        // (the bands' first cells are written behind the tries)
        printf("%d %d %d %d %d", status, parts, lanes, widest, band[PRM_BAND_LO + 1] != 0x55555555);
        for (ll x : W) if (parts) printf(" %lld", x);
        for (int x : bounds) if (parts) printf(" %d", x);
        for (int x : reps) if (parts) printf(" %d", x);
        printf("\n");
        fflush(stdout);
    }
    return 0;
}
