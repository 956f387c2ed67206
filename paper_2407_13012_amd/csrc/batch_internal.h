// Shared by the two halves of the batched engine: batch.hip (C ABI, one
// workgroup per small instance) and batch_many.hip (larger instances, all of
// one size swept together).
#pragma once
#include "qaoa_internal.h"

namespace qk {

constexpr int kMaxP = 16;       // depth limit of the batched engine
constexpr int kMaxPasses = 16;  // passes per mixer layer
constexpr int kMaxBatchN = QAOA_BATCH_MAX_QUBITS;
constexpr int kManyStreams = 3;  // with the small instances' stream one per hardware queue

struct BatchArgs {
    int32_t count;
    int32_t begin, end;     // this launch's range of the processing order
    const int32_t *order;   // processing order (largest n first)
    const int32_t *nq;      // [count] qubits
    const int64_t *eoff;    // [count + 1] edge offsets
    const int32_t *edges;   // [E][2]
    const double *w;        // [E] (NULL: unit weights)
    const double *scale;    // [count] objective scale (1 / sum |w|)
    double *gamma, *beta;   // [count][p] start in, optimum out
    double *e_first;        // [count] E at the start angles
    double *e_last;         // [count] E at the final angles
    int32_t p, steps;
    double lr, b1, b2, eps;
    const Geometry *geo;    // [(kMaxBatchN + 1) * kMaxPasses]
    const int32_t *npass;   // [kMaxBatchN + 1]
    double2 *psi, *lam;     // slot arrays, `slot` amplitudes each
    double *cost;
    uint64_t slot;
    uint32_t *counter;      // this launch's queue counter
    uint64_t *ticks;        // [count][2] device wall clock at an instance's start and end
};

// The instances of one size n > kTileBits (a range of the processing order).
// They run in lockstep: every pass is one launch over the tiles of `cap`
// instances at a time, whose folded vectors, angles and Adam moments are laid
// out one after the other.
struct SizeClass {
    int n = 0;
    int begin = 0, count = 0;  // range of the processing order
    int cap = 0;               // instances at a time
    int stream = 0;
    bool far = false;          // this run's phases may leave the fast range: not run here
    uint64_t M = 0, T = 0;     // stored amplitudes and tiles per instance
    int quad = 0;              // tile bits of the small-tile sweeps (0: the large tiles)
    std::vector<Geometry> geo; // folded passes of one layer
    double2 *psi = nullptr, *lam = nullptr;
    double *cost = nullptr;
    double *parts = nullptr;   // [2p + 1][cap][T]
    double *am = nullptr, *av = nullptr;  // [cap][2p]
    LayerCoef *coef = nullptr; // [cap][p]
    int32_t *step = nullptr;   // [cap] Adam steps done
};

// Size classes of the instances order[0 .. nbig), cut out of `amps` amplitudes
// of vector space; small buffers are counted in *scratch (bytes).  depth[n]: most
// qubits a pass after the first may rotate, which `plans` keep to.
std::vector<SizeClass> make_classes(const std::vector<int32_t> &order, const int32_t *n, int nbig, int p,
                                    uint64_t amps, const std::vector<std::vector<PassPlan>> &plans, const int *depth, size_t *scratch);
// Carves the classes' vectors (from psi, lam, cost) and small buffers (from scratch).
void place_classes(std::vector<SizeClass> &cls, int p, double2 *psi, double2 *lam, double *cost, void *scratch);
// Enqueues the whole optimisation of the classes not marked far on the kManyStreams streams.
hipError_t run_classes(const std::vector<SizeClass> &cls, const BatchArgs &B, hipStream_t *streams);

}  // namespace qk
