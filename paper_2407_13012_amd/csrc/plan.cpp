// Pass planning for the mixer layer (host only).
//
// The mixer prod_j exp(-i b X_j) (Eq. (1)) factorises over qubits and its
// factors commute, so a layer may rotate any group of qubits per sweep over
// the state.  A sweep here is a tiled pass: a workgroup owns 2^TB amplitudes
// whose indices differ only in TB chosen bits (the tile bits; TB = 12 for
// 16-byte amplitudes, 13 for 8-byte ones, 64 KiB either way) and rotates the
// target bits among them.  The plan fixes, for one layer, the tile bits and
// target bits of each pass:
//   * pass 0 rotates a contiguous run of low bits [0, TB - x0) plus x0 high
//     bits, so its global accesses are runs of >= 64 consecutive amplitudes;
//   * passes 1.. keep the S = TB - k lowest bits as non-rotated spectators
//     (runs of 2^S consecutive amplitudes) and rotate k <= 10 further bits,
//     so that runs are >= 64 bytes at either precision;
//   * bits whose stride spans a 2 MiB page (bit >= 17 for 16-byte amplitudes,
//     >= 18 for 8-byte ones) are spread evenly over the passes, since every
//     such target bit doubles the number of pages one tile touches.
#include "qaoa_internal.h"

#include <algorithm>

namespace qk {

namespace {

uint64_t low_mask(int b) { return b >= 64 ? ~0ull : ((1ull << b) - 1ull); }

// Split the set bits of `m` (restricted to [0, n)) into maximal runs of
// consecutive bits, listed in ascending order.
std::vector<std::pair<int, int>> runs_of(uint64_t m, int n)
{
    std::vector<std::pair<int, int>> r;  // (first bit, length)
    int b = 0;
    while (b < n) {
        if (!((m >> b) & 1ull)) {
            ++b;
            continue;
        }
        int e = b;
        while (e < n && ((m >> e) & 1ull)) ++e;
        r.push_back({b, e - b});
        b = e;
    }
    return r;
}

std::vector<PassPlan> plan_simple(int n, int TB, int kmax)
{
    std::vector<PassPlan> out;
    out.push_back({low_mask(TB), low_mask(TB)});
    const int r = n - TB, P = (r + kmax - 1) / kmax;
    int h = TB;
    for (int i = 0; i < P; ++i) {
        const int k = r / P + (i < r % P ? 1 : 0);
        const uint64_t tg = low_mask(k) << h;
        out.push_back({tg | low_mask(TB - k), tg});
        h += k;
    }
    return out;
}

bool plan_ok(int n, int TB, const std::vector<PassPlan> &pl)
{
    uint64_t seen = 0;
    for (const PassPlan &p : pl) {
        if (__builtin_popcountll(p.tile_bits) != std::min(n, TB)) return false;
        if ((p.target_bits & ~p.tile_bits) || (seen & p.target_bits)) return false;
        seen |= p.target_bits;
        Geometry g;
        if (!make_geometry(n, p, &g)) return false;
    }
    return seen == low_mask(n);
}

}  // namespace

// Plan on tiles of 2^TB amplitudes.
static std::vector<PassPlan> plan_tiles(int n, bool c64, int TB, int kmax)
{
    if (n <= TB) return {{low_mask(n), low_mask(n)}};
    const int page = c64 ? 18 : 17;
    const int r = n - TB, P1 = (r + kmax - 1) / kmax;
    std::vector<int> k(P1 + 1), x(P1 + 1, 0), cap(P1 + 1);
    k[0] = TB;
    for (int i = 0; i < P1; ++i) k[i + 1] = r / P1 + (i < r % P1 ? 1 : 0);
    cap[0] = TB - 6;  // pass 0 keeps >= 64 consecutive amplitudes
    for (int i = 1; i <= P1; ++i) cap[i] = k[i];
    int left = std::max(0, n - page);
    while (left > 0) {
        bool moved = false;
        for (int i = 0; i <= P1 && left > 0; ++i)
            if (x[i] < cap[i]) {
                ++x[i];
                --left;
                moved = true;
            }
        if (!moved) break;
    }
    std::vector<PassPlan> out(P1 + 1);
    int nc = TB - x[0];           // next non-crossing bit to hand out
    int cr = std::max(page, TB);  // next crossing bit to hand out
    if (n <= page) cr = n;
    // Crossing bits are handed out in ascending blocks: pass 1 first, then
    // pass 0, then passes 2..  (the order measured fastest at n = 32).
    std::vector<int> order;
    if (P1 >= 1) order.push_back(1);
    order.push_back(0);
    for (int i = 2; i <= P1; ++i) order.push_back(i);
    std::vector<uint64_t> crossing(P1 + 1, 0);
    for (int i : order)
        for (int j = 0; j < x[i]; ++j) crossing[i] |= 1ull << cr++;
    out[0].target_bits = low_mask(TB - x[0]) | crossing[0];
    out[0].tile_bits = out[0].target_bits;
    for (int i = 1; i <= P1; ++i) {
        uint64_t tg = crossing[i];
        for (int j = 0; j < k[i] - x[i]; ++j) tg |= 1ull << nc++;
        out[i].target_bits = tg;
        out[i].tile_bits = tg | low_mask(TB - k[i]);
    }
    if (!plan_ok(n, TB, out)) out = plan_simple(n, TB, kmax);
    return out;
}

std::vector<PassPlan> plan_passes(int n, bool c64, int kmax)
{
    // >= TB - 10 spectator bits: runs of >= 4 (16-byte) or >= 8 (8-byte) amplitudes
    return plan_tiles(n, c64, tile_bits(c64), std::min(std::max(kmax, 1), 10));
}

// Tiles of twice the size where two groups of qubits then make a layer instead of
// three, that is one sweep less per layer and direction of two: n = 23 and 24
// (complex64 24 and 25).  One workgroup fills the LDS of a CU, so its loads, its
// arithmetic and its stores have less beside them to hide in: a sweep takes longer
// per byte (a complex128 backward layer-boundary sweep 3.3 instead of 4.7 TB/s:
// the CUs load, compute and store at the same time), and where no sweep is saved
// the smaller tiles are better.  E + G, p = 4, smaller and large tiles, us:
// complex128 MaxCut n = 23 692 and 540, 24 1340 and 1030, QUBO n = 24 2610 and
// 2056; complex64 MaxCut n = 25 1443 and 1159, QUBO n = 25 2806 and 2276; states
// alone gain as much (n = 25, complex64: 1024 and 869).
int large_tile_bits(int n, bool c64)
{
    const int tb = tile_bits(c64), most = tb + 1 - (c64 ? 3 : 2);  // targets above runs of 64 bytes
    return n - tb > 10 && n - (tb + 1) <= most ? tb + 1 : 0;
}

std::vector<PassPlan> plan_large(int n, bool c64)
{
    const int TB = tile_bits(c64) + 1;
    return plan_tiles(n, c64, TB, TB - (c64 ? 3 : 2));
}

// Two sweeps per layer: the low M bits, then the n - M others over at least 2
// (complex64: 3) spectators, runs of 64 bytes.  M is the smallest of 10, 11, 12
// that leaves room for them.
// Up to 16 MiB of stored state a sweep is bound by the time of one workgroup;
// beyond, by memory, where the large tiles are better (E + G, p = 6, large and
// small tiles, us: complex128 MaxCut n = 14 236 and 110, 17 230 and 122, 20 288
// and 204, 21 (16 MiB) 331 and 269, 22 431 and 447; QUBO n = 20 (16 MiB) 318 and
// 262, 21 425 and 446; complex64 MaxCut n = 21 311 and 222).
int quad_tile_bits(int n, int stored_bits, bool c64)
{
    const int spect = c64 ? 3 : 2;
    if (n <= kSmallBits || stored_bits > (c64 ? 21 : 20)) return 0;
    for (int M = 10; M <= 12; ++M)
        if (n - M <= M - spect && n - M >= M - 8) return M;
    return 0;
}

std::vector<PassPlan> plan_quad(int n, int M)
{
    const int k = n - M;
    return {{low_mask(M), low_mask(M)}, {low_mask(M - k) | (low_mask(k) << M), low_mask(k) << M}};
}

bool make_geometry(int n, const PassPlan &pp, Geometry *g)
{
    *g = Geometry{};
    const auto tr = runs_of(pp.tile_bits, n);
    const auto fr = runs_of(low_mask(n) & ~pp.tile_bits, n);
    if ((int)tr.size() > kTileRuns || (int)fr.size() > kFreeRuns) return false;
    uint32_t local = 0;
    for (size_t i = 0; i < tr.size(); ++i) {
        g->t_src[i] = local;
        g->t_dst[i] = (uint32_t)tr[i].first;
        g->t_len[i] = (uint32_t)tr[i].second;
        for (int j = 0; j < tr[i].second; ++j)
            if ((pp.target_bits >> (tr[i].first + j)) & 1ull) g->tmask |= 1u << (local + j);
        local += (uint32_t)tr[i].second;
    }
    uint32_t t = 0;
    for (size_t i = 0; i < fr.size(); ++i) {
        g->f_src[i] = t;
        g->f_dst[i] = (uint32_t)fr[i].first;
        g->f_len[i] = (uint32_t)fr[i].second;
        t += (uint32_t)fr[i].second;
    }
    g->tbits = local;
    // accesses are coalesced only if the lowest tile bits start at bit 0
    return tr.empty() ? false : tr[0].first == 0;
}

void fold_geometry(int n, const PassPlan &pp, Geometry *g)
{
    g->fold_bit = (uint32_t)(n - 1);
    g->fold = ((pp.tile_bits >> (n - 1)) & 1ull) ? low_mask(n) : 0ull;
}

}  // namespace qk
