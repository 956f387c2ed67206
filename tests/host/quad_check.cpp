// The small-tile plans (qk::plan_quad): for every size and precision that takes
// them the two passes rotate every qubit once, the tiles cover the (folded)
// state, and the tile bits from 8 up are all rotated, which the kernels assume.
#include "qaoa_internal.h"

#include <cstdio>

int main()
{
    int sizes = 0;
    for (int c64 = 0; c64 < 2; ++c64)
        for (int n = 1; n <= 40; ++n)
            for (int fold = 0; fold < 2; ++fold) {
                if (fold && !qk::fold_state(n, c64, true)) continue;
                const int M = qk::quad_tile_bits(n, n - fold, c64);
                if (!M) {
                    // every size between the one-launch states and 16 MiB that two sweeps can cover takes them
                    if (n > qk::kSmallBits && n - fold <= (c64 ? 21 : 20) && n <= (c64 ? 21 : 22)) return std::printf("n=%d c64=%d\n", n, c64), 1;
                    continue;
                }
                ++sizes;
                uint64_t seen = 0;
                for (const qk::PassPlan &p : qk::plan_quad(n, M)) {
                    qk::Geometry g;
                    bool ok = qk::make_geometry(n, p, &g) && (int)g.tbits == M &&
                              (g.tmask >> 8) == ((1u << M) - 1u) >> 8 && !(seen & p.target_bits) &&
                              (p.tile_bits & (c64 ? 7u : 3u)) == (c64 ? 7u : 3u);
                    seen |= p.target_bits;
                    if (fold) qk::fold_geometry(n, p, &g);
                    const uint64_t stored = 1ull << (n - fold);
                    std::vector<unsigned char> at(n <= 18 ? stored : 0, 0);
                    for (uint64_t t = 0; ok && n <= 18 && t < stored >> M; ++t)
                        for (uint32_t e = 0; ok && e < (1u << M); ++e) {
                            const uint64_t a = qk::tile_base(t, g) ^ qk::dep(e, g);
                            ok = a < stored && !at[a]++;
                        }
                    if (!ok) return std::printf("n=%d c64=%d fold=%d M=%d\n", n, c64, fold, M), 1;
                }
                if (seen != (1ull << n) - 1) return std::printf("targets n=%d c64=%d\n", n, c64), 1;
            }
    std::printf("small tiles ok (%d)\n", sizes);
    return 0;
}
