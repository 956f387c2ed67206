// What the library's calls do on the host: which memory they take, which kernels
// they launch and in what order (fake_hip.h).  argv[1] names the check.
#include "fake_hip.h"
#include "qaoa.h"

#include <algorithm>
#include <cmath>

namespace {

const double kGamma[3] = {0.2, 0.3, 0.4}, kBeta[3] = {0.6, 0.5, 0.4};

qaoa_handle ring(int n, int precision = QAOA_C128)
{
    std::vector<int32_t> e;
    for (int i = 0; i < n; ++i) {
        e.push_back(i);
        e.push_back((i + 1) % n);
    }
    qaoa_handle h = nullptr;
    EXPECT(qaoa_create_maxcut(n, n, e.data(), nullptr, precision, nullptr, &h) == QAOA_OK);
    return h;
}

void gradient(qaoa_handle h)
{
    double E, dg[3], db[3];
    EXPECT(qaoa_gradient(h, 3, kGamma, kBeta, &E, dg, db) == QAOA_OK);
}

// A handle's first three results are copied from device memory; its fourth call
// pins memory, once, and before it launches anything.
void pinned_results()
{
    for (int n : {10, 14, 22}) {  // one launch, small tiles, large sweeps
        qaoa_handle h = ring(n);
        const int before = fake().pins;
        for (int k = 0; k < 3; ++k) gradient(h);
        EXPECT(fake().pins == before);
        fake().log.clear();
        gradient(h);
        EXPECT(fake().pins == before + 1 && fake().log.front() == "pin");
        double E;
        gradient(h);
        EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK && qaoa_expectation(h, &E) == QAOA_OK);
        EXPECT(fake().pins == before + 1);
        qaoa_destroy(h);
    }
    // each call takes one result, whatever it computes
    qaoa_handle h = ring(14);
    const int before = fake().pins;
    double E;
    EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK && qaoa_expectation(h, &E) == QAOA_OK);
    gradient(h);
    EXPECT(fake().pins == before);
    fake().log.clear();
    EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK);
    EXPECT(fake().pins == before + 1 && fake().log.front() == "pin");
    qaoa_destroy(h);
}

// Memory that cannot be pinned is not asked for again.
void pinning_refused()
{
    fake().pin_fails = true;
    qaoa_handle h = ring(14);
    const int before = fake().pins;
    for (int k = 0; k < 8; ++k) gradient(h);
    EXPECT(fake().pins == before + 1);
    qaoa_destroy(h);
}

// The allocation of `bytes` bytes, the first a handle made of that size.
const uint8_t *buffer(size_t bytes)
{
    for (const auto &kv : fake().live)
        if (kv.second == bytes) return (const uint8_t *)kv.first;
    EXPECT(!"no such allocation");
    return nullptr;
}

// Whole host arrays of a folded handle: the stored half and its mirror image, in
// pageable and pinned memory at any address, with no device memory to be had.
void host_exports()
{
    for (int n : {14, 18}) {
        for (int prec : {QAOA_C128, QAOA_C64}) {
            const size_t N = (size_t)1 << n, amp = prec == QAOA_C64 ? 8 : 16;
            qaoa_handle h = ring(n, prec);
            std::vector<uint8_t> out(N * 16 + 64);
            const uint8_t *psi = buffer(N / 2 * amp);
            for (int pin = 0; pin < 2; ++pin)
                for (size_t at : {0, 8, 4}) {
                    fake().pinned = pin ? (char *)out.data() : nullptr;
                    fake().pinned_bytes = pin ? out.size() : 0;
                    fake().largest = fake().free_bytes = 0;
                    uint8_t *o = out.data() + at;
                    EXPECT(qaoa_statevector(h, 3, kGamma, kBeta, o, 0) == QAOA_OK);
                    for (size_t z = 0; z < N; ++z)
                        EXPECT(!std::memcmp(o + z * amp, psi + (z < N / 2 ? z : N - 1 - z) * amp, amp));
                    if (prec == QAOA_C128) {
                        const uint8_t *cost = buffer(N / 2 * 8);
                        EXPECT(qaoa_cost_diagonal(h, (double *)o, 0) == QAOA_OK);
                        for (size_t z = 0; z < N; ++z)
                            EXPECT(!std::memcmp(o + z * 8, cost + (z < N / 2 ? z : N - 1 - z) * 8, 8));
                    }
                    fake().largest = ~(size_t)0;
                    fake().free_bytes = 1ull << 40;
                }
            qaoa_destroy(h);
        }
    }
}

// Whole device arrays of a folded handle: its own device's memory is written by a
// kernel, memory of another device or unknown to the runtime only by copies.
void device_exports()
{
    for (int prec : {QAOA_C128, QAOA_C64}) {
        const int n = 14;
        const size_t N = (size_t)1 << n, amp = prec == QAOA_C64 ? 8 : 16;
        qaoa_handle h = ring(n, prec);
        const uint8_t *psi = buffer(N / 2 * amp), *cost = prec == QAOA_C128 ? buffer(N / 2 * 8) : nullptr;
        const std::vector<uint8_t> was(psi, psi + N / 2 * amp);
        for (int kind = 0; kind < 3; ++kind) {
            void *out = nullptr;
            if (kind < 2) EXPECT(hipMalloc(&out, N * 16 + 16) == hipSuccess);
            else out = std::malloc(N * 16 + 16);
            if (kind == 1) fake().owner[out] = 1;
            uint8_t *o = (uint8_t *)out + 16;
            fake().log.clear();
            EXPECT(qaoa_statevector(h, 3, kGamma, kBeta, o, 1) == QAOA_OK);
            for (size_t z = 0; z < N; ++z)
                EXPECT(!std::memcmp(o + z * amp, &was[(z < N / 2 ? z : N - 1 - z) * amp], amp));
            EXPECT(!std::memcmp(psi, was.data(), was.size()));
            if (cost) {
                EXPECT(qaoa_cost_diagonal(h, (double *)o, 1) == QAOA_OK);
                for (size_t z = 0; z < N; ++z) EXPECT(!std::memcmp(o + z * 8, cost + (z < N / 2 ? z : N - 1 - z) * 8, 8));
            }
            EXPECT(launches("k_unfold_words") == (kind == 0 ? (cost ? 2 : 1) : 0));
            fake().owner.erase(out);
            if (kind < 2) EXPECT(hipFree(out) == hipSuccess);
            else std::free(out);
        }
        qaoa_destroy(h);
    }
}

// Free memory is compared with what a handle allocates: half of the state for a
// folded one (16 + 8 bytes per amplitude, the adjoint vector 16 more), all of it
// for a polynomial.
void memory_checks()
{
    const int n = 20;
    const size_t half = (size_t)1 << (n - 1), room = 2 << 20;
    fake().free_bytes = half * 24 + room;
    qaoa_handle h = ring(n);
    const uint64_t mask = 3;
    const double w = 1.0;
    qaoa_handle whole = nullptr;
    EXPECT(qaoa_create_poly(n, 1, &mask, &w, 0.0, QAOA_C128, nullptr, &whole) == QAOA_ERR_OUT_OF_MEMORY && !whole);
    double E, dg[3], db[3];
    fake().free_bytes = half * 16 - 1;
    EXPECT(qaoa_gradient(h, 3, kGamma, kBeta, &E, dg, db) == QAOA_ERR_OUT_OF_MEMORY);
    fake().free_bytes = half * 16;
    gradient(h);
    qaoa_destroy(h);
    fake().free_bytes = half * 24;
    std::vector<int32_t> e = {0, 1};
    EXPECT(qaoa_create_maxcut(n, 1, e.data(), nullptr, QAOA_C128, nullptr, &h) == QAOA_ERR_OUT_OF_MEMORY);
}

// A handle is usable after an allocation that failed, its own or another object's.
void failed_allocations()
{
    qaoa_handle h = ring(20);
    double E, dg[3], db[3];
    fake().largest = (size_t)1 << 20;
    EXPECT(qaoa_gradient(h, 3, kGamma, kBeta, &E, dg, db) == QAOA_ERR_OUT_OF_MEMORY);
    EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK);
    qaoa_mpnn m = nullptr;
    fake().largest = 0;
    EXPECT(qaoa_mpnn_create(4, &m) == QAOA_ERR_DEVICE);
    EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK);
    const int32_t n = 9, edge[2] = {0, 1};
    const int64_t off[2] = {0, 1};
    qaoa_batch b = nullptr;
    EXPECT(qaoa_batch_create(1, &n, off, edge, nullptr, 1, nullptr, &b) == QAOA_ERR_DEVICE);
    EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK);
    fake().largest = ~(size_t)0;
    gradient(h);
    qaoa_destroy(h);
}

// Shots to device memory return once the total is known, while they run: an event
// behind the scan.  Shots to host memory wait for the stream, with no event.
void sample_waits()
{
    qaoa_handle h = ring(14);
    for (int k = 0; k < 4; ++k) gradient(h);
    double E, cost[8];
    uint64_t z[8];
    EXPECT(qaoa_evaluate(h, 3, kGamma, kBeta, &E) == QAOA_OK);
    for (int device = 0; device < 2; ++device) {
        fake().log.clear();
        EXPECT(qaoa_sample(h, 8, 1, z, cost, device) == QAOA_OK);
        EXPECT(launches("event") == device && launches("k_shots") == 1);
        if (device) EXPECT(fake().log[fake().log.size() - 2] == "event");
    }
    qaoa_destroy(h);
}

// A batch of rings of the given sizes and one weight for all edges of each.
struct Batch {
    std::vector<int32_t> n, edges;
    std::vector<int64_t> off{0};
    std::vector<double> w;
    qaoa_batch_options o{100, 0.05, 0.9, 0.999, 1e-8, 0, 10, 1, 0, {}, 0};
    qaoa_batch b = nullptr;
    Batch(const std::vector<int> &sizes, const std::vector<double> &weights)
    {
        for (size_t k = 0; k < sizes.size(); ++k) {
            n.push_back(sizes[k]);
            for (int i = 0; i < sizes[k]; ++i) {
                edges.push_back(i);
                edges.push_back((i + 1) % sizes[k]);
                w.push_back(weights[k]);
            }
            off.push_back((int64_t)w.size());
        }
    }
    qaoa_status create()
    {
        return qaoa_batch_create((int32_t)n.size(), n.data(), off.data(), edges.data(), w.data(), 2, &o, &b);
    }
    // the launches of one run from these gammas (both layers), 0.3 where none is given
    void run(std::vector<double> gamma = {})
    {
        std::vector<double> g;
        for (size_t k = 0; k < n.size(); ++k) g.insert(g.end(), 2, k < gamma.size() ? gamma[k] : 0.3);
        std::vector<double> og(g), ob(g);
        fake().log.clear();
        EXPECT(qaoa_batch_run(b, g.data(), g.data(), og.data(), ob.data(), nullptr, nullptr) == QAOA_OK);
    }
    ~Batch() { qaoa_batch_destroy(b); }
};

// A batch whose slots fit, but not what the size classes keep beside them, runs as
// one persistent launch.
void batch_without_class_scratch()
{
    const std::vector<int> sizes = {14, 13, 9};
    const std::vector<double> w = {1.0, 1.0, 1.0};
    size_t all = 0;
    {
        Batch b(sizes, w);
        b.o.use_graph = 0;
        b.o.steps = 1;
        EXPECT(b.create() == QAOA_OK);
        all = fake().taken;
        b.run();
        EXPECT(launches("k_many_adam") == 2 && launches("k_batch") == 1);
    }
    for (int graph : {0, 1}) {
        Batch b(sizes, w);
        b.o.use_graph = graph;
        fake().budget = all - 1;
        fake().log.clear();
        EXPECT(b.create() == QAOA_OK);
        EXPECT(graph == 0 || launches("k_batch") == 1);  // captured
        b.run();
        EXPECT(launches("k_many") == 0 && launches("k_batch") == (graph ? 0 : 1));
    }
    fake().budget = ~(size_t)0;
}

// What `steps` steps of Adam can move an angle by at most.
double reach(const qaoa_batch_options &o)
{
    double s = 0.0;
    const double r = o.beta1 * o.beta1 / o.beta2;
    for (int t = 1; t <= o.steps; ++t)
        s += o.lr * (1 - o.beta1) / (1 - std::pow(o.beta1, t)) *
             std::sqrt((1 - std::pow(o.beta2, t)) * (1 - std::pow(r, t)) / ((1 - o.beta2) * (1 - r)));
    return s;
}

// Instances run in their size class while |gamma| sum|w| stays below 5e5 over the
// start angle 0.3 and all that Adam can add.
void batch_phase_bound()
{
    for (int steps : {0, 1, 100, 4096, 6000}) {
        for (double side : {0.99, 1.001}) {
            Batch b({14}, {0.0});
            b.o.steps = steps;
            b.o.lr = 1e-3;
            const double weight = side * 5e5 / (0.3 + reach(b.o)) / 14;
            std::fill(b.w.begin(), b.w.end(), weight);
            EXPECT(b.create() == QAOA_OK);
            b.run();
            EXPECT(launches("k_many_adam") == (side < 1.0 ? steps : 0));
            EXPECT(launches("k_many_final") == (side < 1.0 ? 1 : 0));
            EXPECT((launches("k_batch") > 0) == (side > 1.0));
        }
    }
}

// Only the sizes of which an instance's own phases may leave the range go to the
// persistent launch, neighbours in size together, after the other sizes.
void batch_far_sizes()
{
    const double heavy = 1e6;
    const struct {
        std::vector<int> n;
        std::vector<double> w, gamma;
        int classes, queues;  // size classes run, persistent launches
    } cases[] = {
        {{16, 15, 14, 9}, {1, heavy, 1, 1}, {}, 2, 2},       // one-tile, then n = 15
        {{16, 15, 14, 9}, {heavy, heavy, 1, 1}, {}, 1, 2},   // 16 and 15 in one launch
        {{16, 15, 14, 9}, {heavy, 1, heavy, 1}, {}, 1, 3},
        {{16, 15, 14, 9}, {heavy, heavy, heavy, 1}, {}, 0, 1},  // all in one launch
        {{15, 14, 15}, {1, 1, heavy}, {}, 1, 1},             // a size with one such instance
        {{15, 14}, {heavy, 1}, {1e-9, 1e3}, 2, 0},           // its own angles count
    };
    for (const auto &c : cases) {
        Batch b(c.n, c.w);
        b.o.steps = c.gamma.empty() ? 2 : 0;
        b.o.use_graph = 0;
        EXPECT(b.create() == QAOA_OK);
        for (int rep = 0; rep < 2; ++rep) {
            b.run(c.gamma);
            EXPECT(launches("k_many_final") == c.classes && launches("k_batch") == c.queues);
            b.run({1e12, 1e12, 1e12, 1e12});  // every size
            EXPECT(launches("k_many") == 0 && launches("k_batch") == 1);
        }
    }
}

// A batch has its own stream and one for each size class, up to three.
void batch_streams()
{
    const std::vector<std::vector<int>> batches = {{12, 9}, {13, 13, 9}, {14, 13}, {16, 15, 14, 13, 13, 4}};
    const int more[] = {0, 1, 2, 3};
    for (size_t k = 0; k < batches.size(); ++k) {
        const int before = fake().streams;
        Batch b(batches[k], std::vector<double>(batches[k].size(), 1.0));
        b.o.steps = 1;
        EXPECT(b.create() == QAOA_OK && fake().streams == before + 1 + more[k]);
        b.run();
        EXPECT(fake().streams == before + 1 + more[k]);
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> checks = {
        {"pinned_results", pinned_results},
        {"pinning_refused", pinning_refused},
        {"host_exports", host_exports},
        {"device_exports", device_exports},
        {"memory_checks", memory_checks},
        {"failed_allocations", failed_allocations},
        {"sample_waits", sample_waits},
        {"batch_without_class_scratch", batch_without_class_scratch},
        {"batch_phase_bound", batch_phase_bound},
        {"batch_far_sizes", batch_far_sizes},
        {"batch_streams", batch_streams},
    };
    const auto it = checks.find(argc > 1 ? argv[1] : "");
    EXPECT(it != checks.end());
    it->second();
    EXPECT(fake().live.empty());
    std::printf("%s ok\n", argv[1]);
    return 0;
}
