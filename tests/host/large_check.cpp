// The large-tile plans (qk::plan_large): the sizes that take them are those of
// which two groups of qubits make a layer on large tiles and three on the others;
// the passes rotate every qubit once, are of the spectator classes that have
// kernels, and every tile stays inside the (folded) state, the tiles of sampled
// neighbourhoods being disjoint.
#include "qaoa_internal.h"

#include <cstdio>
#include <set>

int main()
{
    int sizes = 0;
    for (int c64 = 0; c64 < 2; ++c64)
        for (int n = 1; n <= 40; ++n) {
            const int M = qk::large_tile_bits(n, c64), least = c64 ? 3 : 2;
            const bool want = qk::plan_passes(n, c64).size() == 3 && n <= 2 * (qk::tile_bits(c64) + 1) - least;
            if ((M != 0) != want || (M && M != qk::tile_bits(c64) + 1)) return std::printf("size n=%d c64=%d\n", n, c64), 1;
            if (!M) continue;
            ++sizes;
            const std::vector<qk::PassPlan> plan = qk::plan_large(n, c64);
            uint64_t seen = 0;
            if (plan.size() != 2) return std::printf("passes n=%d c64=%d\n", n, c64), 1;
            for (int fold = 0; fold < 2; ++fold)
                for (const qk::PassPlan &p : plan) {
                    qk::Geometry g;
                    bool ok = qk::make_geometry(n, p, &g) && (int)g.tbits == M;
                    const int S = __builtin_ctz(g.tmask);
                    ok = ok && g.tmask == ((1u << M) - 1u) - ((1u << S) - 1u) && (S == 0 || S == least || S == least + 1);
                    // runs of 64 amplitudes or more exactly in class 0 (streaming accesses)
                    ok = ok && g.t_dst[0] == 0 && (g.t_len[0] >= 6) == (S == 0);
                    if (!fold) {
                        ok = ok && !(seen & p.target_bits);
                        seen |= p.target_bits;
                    } else {
                        qk::fold_geometry(n, p, &g);
                    }
                    const uint64_t stored = 1ull << (n - fold), tiles = stored >> M;
                    std::set<uint64_t> at;
                    for (uint64_t t : {(uint64_t)0, (uint64_t)1, tiles / 2, tiles - 1})
                        for (uint32_t e = 0; ok && e < (1u << M); ++e) {
                            const uint64_t a = qk::tile_base(t, g) ^ qk::dep(e, g);
                            ok = a < stored && at.insert(a).second;
                        }
                    if (!ok) return std::printf("n=%d c64=%d fold=%d\n", n, c64, fold), 1;
                }
            if (seen != (1ull << n) - 1) return std::printf("targets n=%d c64=%d\n", n, c64), 1;
        }
    std::printf("large tiles ok (%d)\n", sizes);
    return 0;
}
