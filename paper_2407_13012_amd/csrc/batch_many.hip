// Batched engine, instances of more than one tile (n > 12): all instances of
// one size run in lockstep, one launch per pass over the tiles of all of them.
//
// A workgroup that runs such an instance by itself streams every sweep of it
// through one compute unit: an n = 20 instance takes 38 ms per Adam step beside
// 47 others (48 ms beside 511) and the batch ends with its last large instances
// on a nearly idle card.  Swept together, a pass of one n = 20 instance is 128
// workgroups, and the kernels are those of the single-instance path, compiled
// per spectator class, or on small tiles.  The angles stay on the device: k_many_adam sums the
// partials of a step, updates the angles and leaves the rotations' coefficients
// for the next step's passes.  Sizes are independent of each other and run on
// three streams.  Measured (p = 4, n ~ U{10..20}): 48 graphs x 8 steps
// 325 -> 4.7-5.6 ms, 1024 graphs x 3 steps 206 -> 25-27 ms (there at 5.5 TB/s;
// fewer instances at a time, so that their vectors stay in the last-level cache,
// are slower: 28.0 ms with 192 MB per size, 33.8 with 64 MB).
//
// The instances are MaxCut, so their states are kept folded (fold_state), and
// X on every qubit is the identity on them: beta is reduced to [-pi/4, pi/4],
// where every rotation has the tan form.
#include "batch_internal.h"
#include "tile_device.h"

#include <algorithm>
#include <cmath>
#include <numeric>

namespace qk {
namespace {

constexpr int kAdamThreads = 512;

__device__ __forceinline__ LayerCoef layer_coef(double gamma, double beta)
{
    // exp(-i (b + pi/2) X) = exp(-i b X) (-i X): quarter turns only change a
    // global phase of a state with psi(z) = psi(~z)
    const double k = rint(beta * 0x1.45f306dc9c883p-1);  // 2 / pi
    double r = fma(-k, 0x1.921fb54442d18p+0, beta);       // pi / 2, head and tail
    r = fma(-k, 0x1.1a62633145c07p-54, r);
    double s, c;
    sincos(r, &s, &c);
    return {gamma, s / c, c};
}

// State of a chunk of instances at their start angles: one workgroup each.
__global__ __launch_bounds__(64) void k_many_start(BatchArgs B, int begin, double *am, double *av, LayerCoef *coef,
                                                   int32_t *step)
{
    const int y = blockIdx.x, tid = threadIdx.x, p = B.p;
    const int64_t i = B.order[begin + y];
    if (tid == 0) {
        B.ticks[2 * i] = wall_clock64();
        step[y] = 0;
    }
    if (tid < 2 * p) {
        am[(int64_t)y * 2 * p + tid] = 0.0;
        av[(int64_t)y * 2 * p + tid] = 0.0;
    }
    if (tid < p) coef[(int64_t)y * p + tid] = layer_coef(B.gamma[i * p + tid], B.beta[i * p + tid]);
}

// Folded cost diagonals: the weights of the cut edges of z, added in edge order.
// Thread entries are z = tile * 4096 + r * 256 + thread; an edge with no end in
// bits 8..11 is cut for all 16 or for none.  Adding -0.0 leaves a sum as it is.
__global__ __launch_bounds__(kThreads) void k_many_cost(BatchArgs B, int begin, double *cost, uint64_t M)
{
    const int y = blockIdx.y;
    const int i = B.order[begin + y];
    const int64_t e0 = B.eoff[i], e1 = B.eoff[i + 1];
    const uint32_t z0 = blockIdx.x * (uint32_t)kTile + threadIdx.x;  // n <= 24
    double acc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0;
    for (int64_t k = e0; k < e1; ++k) {
        const int u = B.edges[2 * k], v = B.edges[2 * k + 1];
        const double w = B.w ? B.w[k] : 1.0;
        const uint32_t m = (1u << u) ^ (1u << v);
        const bool cut = ((z0 >> u) ^ (z0 >> v)) & 1u;
        const double w0 = cut ? w : -0.0, w1 = cut ? -0.0 : w;
        if (!(m & 0xF00u)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += w0;
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += (popc(((uint32_t)r << 8) & m) & 1) ? w1 : w0;
        }
    }
    double *c = cost + (uint64_t)y * M;
#pragma unroll
    for (int r = 0; r < 16; ++r) c[z0 + 256u * r] = acc[r];
}

// Sum of one slot's partials of an instance by one wave, in fixed order.
__device__ __forceinline__ double slot_sum(const double *x, uint64_t T)
{
    double s = 0.0;
    for (uint64_t t = threadIdx.x & 63u; t < T; t += 64) s += x[t];
    return 2.0 * wave_sum(s);  // the partials are those of half the state
}

// One Adam step of every instance of the chunk (one workgroup each) from its
// partial sums: slot 0 E, 1 .. p the <lam|X|phi>, p+1 .. 2p the <lam|C|phi> terms.
__global__ __launch_bounds__(kAdamThreads) void k_many_adam(BatchArgs B, int begin, int cap, const double *parts,
                                                            uint64_t T, double *am, double *av, LayerCoef *coef,
                                                            int32_t *step)
{
    __shared__ double sum[2 * kMaxP + 1], th[2 * kMaxP];
    const int y = blockIdx.x, tid = threadIdx.x, p = B.p;
    const int64_t i = B.order[begin + y];
    for (int s = tid >> 6; s <= 2 * p; s += kAdamThreads / 64) {
        const double v = slot_sum(parts + ((uint64_t)s * cap + y) * T, T);
        if ((tid & 63) == 0) sum[s] = v;
    }
    __syncthreads();
    const int t = step[y];
    if (tid < 2 * p) {
        const int l = tid < p ? tid : tid - p;
        const double g = B.scale[i] * (2.0 * (tid < p ? sum[1 + p + l] : sum[1 + l]));
        double *a = am + (int64_t)y * 2 * p + tid, *v = av + (int64_t)y * 2 * p + tid;
        const double a1 = B.b1 * *a + (1.0 - B.b1) * g;
        const double v1 = B.b2 * *v + (1.0 - B.b2) * g * g;
        *a = a1;
        *v = v1;
        const double mh = a1 / (1.0 - pow(B.b1, (double)(t + 1)));
        const double vh = v1 / (1.0 - pow(B.b2, (double)(t + 1)));
        double *x = (tid < p ? B.gamma : B.beta) + i * p + l;
        th[tid] = *x + B.lr * mh / (sqrt(vh) + B.eps);
        *x = th[tid];
    }
    __syncthreads();
    if (tid < p) coef[(int64_t)y * p + tid] = layer_coef(th[tid], th[p + tid]);
    if (tid == 0) {
        if (t == 0) B.e_first[i] = sum[0];
        step[y] = t + 1;
    }
}

// E at the final angles.
__global__ __launch_bounds__(64) void k_many_final(BatchArgs B, int begin, const double *parts, uint64_t T,
                                                   const int32_t *step)
{
    const int y = blockIdx.x;
    const int64_t i = B.order[begin + y];
    const double E = slot_sum(parts + (uint64_t)y * T, T);
    if (threadIdx.x == 0) {
        if (step[y] == 0) B.e_first[i] = E;
        B.e_last[i] = E;
        B.ticks[2 * i + 1] = wall_clock64();
    }
}

// ------------------------------------------------------------------ schedule

// Passes of one class's chunk of `count` instances on one stream; the schedule
// is the single-instance gradient's (forward, turn, backward, layers visiting
// their groups in alternating order so that neighbours share a sweep).
struct Chunk {
    const SizeClass &c;
    const BatchArgs &B;
    int begin;       // of the processing order
    unsigned count;
    hipStream_t s;

    int group(int l, int idx) const
    {
        const int P = (int)c.geo.size();
        return l % 2 == 0 ? idx : P - 1 - idx;
    }
    double *slot(int k) const { return c.parts + (uint64_t)k * c.cap * c.T; }
    double *slotB(int l) const { return slot(1 + l); }
    double *slotG(int l) const { return slot(1 + B.p + l); }

    hipError_t pass(int mode, int gi, int flags, int layer, int layer2, int layer_phase, double *pe = nullptr,
                    double *pb = nullptr, double *pg = nullptr, double *pb2 = nullptr) const
    {
        PassArgs a{};
        a.psi = c.psi;
        a.lam = c.lam;
        a.cost = c.cost;
        a.geo = c.geo[gi];
        // nontemporal for runs of >= 64 amplitudes, as in the single-instance passes
        a.flags = flags | (a.geo.t_dst[0] == 0 && a.geo.t_len[0] >= 6 ? kStream : 0);
        a.xcd_g = xcd_group_bits(c.T, 4);
        a.amp0 = 1.0 / std::sqrt((double)(2 * c.M));
        a.part_e = pe;
        a.part_b = pb;
        a.part_g = pg;
        a.part_b2 = pb2;
        const ManyArgs m{c.coef, c.M, c.T, B.p, layer, layer2, layer_phase};
        return c.quad ? launch_many_quad(mode, c.quad, a, m, c.T, count, s) : launch_many(mode, a, m, c.T, count, s);
    }

    // Layers forward; grad: without the last layer's last group (the turn pass).
    hipError_t forward(bool grad) const
    {
        const int P = (int)c.geo.size(), p = B.p;
        for (int l = 0; l < p; ++l)
            for (int idx = 0; idx < P; ++idx) {
                if (l > 0 && idx == 0) continue;  // shared with layer l - 1's last group
                const bool last = idx == P - 1;
                hipError_t e;
                if (last && l == p - 1) {
                    if (grad) break;
                    e = pass(kFwd, group(l, idx), kEOut, l, l, l, slot(0));
                } else if (last) {
                    e = pass(kFwdFuse, group(l, idx), 0, l, l + 1, l + 1);
                } else {
                    e = pass(kFwd, group(l, idx), l == 0 && idx == 0 ? kInit | kPhaseIn : 0, l, l, l);
                }
                if (e != hipSuccess) return e;
            }
        return hipSuccess;
    }

    hipError_t start() const
    {
        hipLaunchKernelGGL(k_many_start, dim3(count), dim3(64), 0, s, B, begin, c.am, c.av, c.coef, c.step);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_many_cost, dim3((unsigned)(c.M >> kTileBits), count), dim3(kThreads), 0, s, B, begin, c.cost, c.M);
        return hipGetLastError();
    }

    hipError_t step() const
    {
        const int P = (int)c.geo.size(), p = B.p;
        hipError_t e = forward(true);
        if (e != hipSuccess) return e;
        if ((e = pass(kTurn, group(p - 1, P - 1), 0, p - 1, p - 1, p - 1, slot(0), slotB(p - 1))) != hipSuccess) return e;
        for (int l = p - 1; l >= 0; --l)
            for (int idx = P - 1; idx >= 0; --idx) {
                if (idx == P - 1) continue;  // undone by the turn or by layer l + 1's first group
                const int gi = group(l, idx);
                const int noPhi = !c.quad && (P > 2 ? l == 0 && idx == 1 : l == 1 && idx == 0) ? kNoPhi : 0;
                if (idx > 0) e = pass(kBwd, gi, kBetaAcc | noPhi, l, l, l, nullptr, slotB(l));
                else if (l > 0) e = pass(kBwdFuse, gi, kBetaAcc | noPhi, l, l - 1, l, nullptr, slotB(l), slotG(l), slotB(l - 1));
                else e = pass(c.quad ? kBwd : kBwdFirst, gi, kBetaAcc | kPhaseOut | kNoStore, 0, 0, 0, nullptr, slotB(0), slotG(0));
                if (e != hipSuccess) return e;
            }
        hipLaunchKernelGGL(k_many_adam, dim3(count), dim3(kAdamThreads), 0, s, B, begin, c.cap,
                           (const double *)c.parts, c.T, c.am, c.av, c.coef, c.step);
        return hipGetLastError();
    }

    hipError_t finish() const
    {
        hipError_t e = forward(false);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_many_final, dim3(count), dim3(64), 0, s, B, begin, (const double *)c.parts, c.T,
                           (const int32_t *)c.step);
        return hipGetLastError();
    }
};

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t class_scratch(const SizeClass &c, int p)
{
    return up256((size_t)(2 * p + 1) * c.cap * c.T * 8) + 2 * up256((size_t)c.cap * 2 * p * 8) +
           up256((size_t)c.cap * p * sizeof(LayerCoef)) + up256((size_t)c.cap * 4);
}

}  // namespace

std::vector<SizeClass> make_classes(const std::vector<int32_t> &order, const int32_t *n, int nbig, int p,
                                    uint64_t amps, const std::vector<std::vector<PassPlan>> &plans, const int *depth, size_t *scratch)
{
    std::vector<SizeClass> cls;
    for (int k = 0; k < nbig; ++k) {
        const int m = n[order[k]];
        if (cls.empty() || cls.back().n != m) {
            SizeClass c;
            c.n = m;
            c.begin = k;
            c.M = 1ull << (m - 1);
            cls.push_back(c);
        }
        ++cls.back().count;
    }
    // One instance of every class fits (their vectors sum to less than one
    // whole state of the largest size); the rest goes to the classes in turn,
    // the smallest sizes first, whose sweeps fill the card least.
    uint64_t left = amps;
    for (SizeClass &c : cls) {
        c.cap = 1;
        left -= c.M;
    }
    for (auto it = cls.rbegin(); it != cls.rend(); ++it) {
        SizeClass &c = *it;
        const uint64_t more = std::min<uint64_t>({(uint64_t)c.count - 1, left / c.M, 65534});
        c.cap += (int)more;
        left -= more * c.M;
    }
    // Small tiles while all that runs together makes up at most the 16 MiB up to
    // which one state takes them, and the depth asked for allows their two passes.
    // Beside larger classes, which fill the card, only classes of up to 2 MiB gain
    // (48 graphs, n = 10 .. 20: 6.58 ms with none on small tiles, 5.13 with classes
    // of up to 2 MiB, 5.32 with 8, 5.45 with 32).
    uint64_t together = 0;
    for (const SizeClass &c : cls) together += (uint64_t)c.cap * c.M;
    const uint64_t most = together <= (1ull << 20) ? 1ull << 20 : 1ull << 17;
    for (SizeClass &c : cls) {
        c.quad = (uint64_t)c.cap * c.M <= most ? quad_tile_bits(c.n, c.n - 1, false) : 0;
        if (c.quad && c.n - c.quad > depth[c.n]) c.quad = 0;
        c.T = c.M >> (c.quad ? c.quad : kTileBits);
        for (const PassPlan &pp : c.quad ? plan_quad(c.n, c.quad) : plans[c.n]) {
            Geometry g;
            make_geometry(c.n, pp, &g);
            fold_geometry(c.n, pp, &g);
            c.geo.push_back(g);
        }
    }
    // three streams, the most work first to the least loaded: a sweep costs its
    // traffic (440 B per stored amplitude and step) or a launch's latency
    std::vector<size_t> by(cls.size());
    std::iota(by.begin(), by.end(), (size_t)0);
    auto cost = [&](const SizeClass &c) {
        const double sweeps = 2.0 * p * (double)c.geo.size();
        return ((c.count + c.cap - 1) / c.cap) * sweeps * 1e-5 + (double)c.count * (double)c.M * 440.0 * p / 4 / 5e12;
    };
    std::stable_sort(by.begin(), by.end(), [&](size_t a, size_t b) { return cost(cls[a]) > cost(cls[b]); });
    double load[kManyStreams] = {};
    for (size_t k : by) {
        const int s = (int)(std::min_element(load, load + kManyStreams) - load);
        cls[k].stream = s;
        load[s] += cost(cls[k]);
    }
    *scratch = 0;
    for (const SizeClass &c : cls) *scratch += class_scratch(c, p);
    return cls;
}

void place_classes(std::vector<SizeClass> &cls, int p, double2 *psi, double2 *lam, double *cost, void *scratch)
{
    char *b = (char *)scratch;
    auto take = [&](size_t bytes) {
        void *r = b;
        b += up256(bytes);
        return r;
    };
    uint64_t o = 0;
    for (SizeClass &c : cls) {
        c.psi = psi + o;
        c.lam = lam + o;
        c.cost = cost + o;
        o += (uint64_t)c.cap * c.M;
        c.parts = (double *)take((size_t)(2 * p + 1) * c.cap * c.T * 8);
        c.am = (double *)take((size_t)c.cap * 2 * p * 8);
        c.av = (double *)take((size_t)c.cap * 2 * p * 8);
        c.coef = (LayerCoef *)take((size_t)c.cap * p * sizeof(LayerCoef));
        c.step = (int32_t *)take((size_t)c.cap * 4);
    }
}

hipError_t run_classes(const std::vector<SizeClass> &cls, const BatchArgs &B, hipStream_t *streams)
{
    // one unit (start, a step, the final E) of every stream's current class in turn
    struct At {
        size_t k = 0;   // class
        int done = 0;   // instances of it finished
        int unit = -1;  // -1 start, 0 .. steps - 1, steps: final
    } at[kManyStreams];
    for (bool any = true; any;) {
        any = false;
        for (int s = 0; s < kManyStreams; ++s) {
            At &a = at[s];
            while (a.k < cls.size() && (cls[a.k].stream != s || cls[a.k].far)) ++a.k;
            if (a.k == cls.size()) continue;
            any = true;
            const SizeClass &c = cls[a.k];
            const Chunk ch{c, B, c.begin + a.done, (unsigned)std::min(c.cap, c.count - a.done), streams[s]};
            const hipError_t e = a.unit < 0 ? ch.start() : a.unit < B.steps ? ch.step() : ch.finish();
            if (e != hipSuccess) return e;
            if (++a.unit > B.steps) {
                a.unit = -1;
                a.done += (int)ch.count;
                if (a.done >= c.count) {
                    ++a.k;
                    a.done = 0;
                }
            }
        }
    }
    return hipSuccess;
}

}  // namespace qk
