// Folded states (qk::fold_geometry) against the whole ones, for every pass of
// every plan (both precisions, some caps on a later pass's qubits): the tiles a
// folded pass runs (the first half) visit each stored amplitude exactly once,
// each at the place of its index z or, for z with bit n-1 set, of ~z, and the
// partner of an amplitude across a rotated bit is at its stored place too.
// Sizes up to 2^16 are checked in full, larger ones on tiles spread over the range.
#include "qaoa_internal.h"

#include <cstdio>
#include <vector>

static uint64_t stored(uint64_t z, int n) { return (z >> (n - 1)) & 1 ? z ^ ((1ull << n) - 1) : z; }

int main()
{
    long passes = 0;
    for (int c64 = 0; c64 < 2; ++c64)
        for (int n = qk::tile_bits(c64) + 1; n <= 34; ++n)
            for (int kmax = 1; kmax <= 10; kmax += 3) {
                if (!qk::fold_state(n, c64, true) || qk::fold_state(n, c64, false)) return 1;
                const int TB = qk::tile_bits(c64);
                const uint64_t half = 1ull << (n - 1), T = 1ull << (n - 1 - TB);
                const bool all = n <= 16;
                for (const qk::PassPlan &p : qk::plan_passes(n, c64 != 0, kmax)) {
                    qk::Geometry whole, g;
                    qk::make_geometry(n, p, &whole);
                    qk::make_geometry(n, p, &g);
                    qk::fold_geometry(n, p, &g);
                    std::vector<unsigned char> seen(all ? half : 0, 0);
                    const uint64_t step = all ? 1 : T / 2 + 1;
                    for (uint64_t t = 0; t < T; t += step) {
                        const uint64_t base = qk::tile_base(t, g);
                        for (uint32_t e = 0; e < (1u << TB); ++e) {
                            const uint64_t z = qk::tile_base(t, whole) | qk::dep(e, whole);
                            const uint64_t a = base ^ qk::dep(e, g);
                            // the address is linear over XOR in e: thread part, register part
                            const uint64_t b = base ^ qk::dep(e & 0x3f5u, g) ^ qk::dep(e & ~0x3f5u, g);
                            bool ok = a < half && a == stored(z, n) && a == b;
                            for (int j = 0; j < TB && ok; ++j) {
                                const uint64_t zj = qk::tile_base(t, whole) | qk::dep(e ^ (1u << j), whole);
                                ok = (base ^ qk::dep(e ^ (1u << j), g)) == stored(zj, n);
                            }
                            if (all && ok) ok = !seen[a]++;
                            if (!ok) {
                                std::printf("n=%d c64=%d kmax=%d tile %llu element %u\n", n, c64, kmax,
                                            (unsigned long long)t, e);
                                return 1;
                            }
                        }
                    }
                    for (unsigned char s : seen)
                        if (!s) return std::printf("n=%d c64=%d kmax=%d: amplitude not visited\n", n, c64, kmax), 1;
                    ++passes;
                }
            }
    std::printf("folded passes ok (%ld)\n", passes);
    return 0;
}
