// gfx950 kernels of the QAOA statevector path.
//
// Streaming pass kernel (k_pass)
//   The mixer U_M(b) = prod_j exp(-i b X_j) is a product of commuting
//   single-qubit rotations (Eq. (1); Sec. IV-B applies them gate by gate).
//   Instead of one full-state sweep per qubit, a pass loads a tile of 2^TB
//   amplitudes whose index bits cover a group of qubits, applies every rotation
//   of that group in registers, and writes the tile back once (TB = 12 for
//   complex128, 13 for complex64: 64 KiB of state per tile either way).  A
//   tile is the set of indices with bits [0,S) and [h,h+k) free (S + k = TB);
//   the other n-TB bits are fixed by the workgroup.  Each thread holds 16
//   amplitudes (256 threads for complex128, 512 for complex64); three register
//   arrangements (A, B, C) each put four different tile bits into the register
//   index, and two LDS transposes move between them, so every tile bit up to
//   11 is a register bit once.  For TB = 12:
//     A: lane = bits 0-5,        reg = bits 6-9,         wave = bits 10-11
//     B: reg = bits 0-3,         lane = bits 4-9,        wave = bits 10-11
//     C: lane = bits 0-3,6,7,    reg = bits 4,5,10,11,   wave = bits 8-9
//   For TB = 13 bit 12 is a third wave bit in A and C and lane bit 1 in B, where
//   its rotation pairs each lane with the one 2 away (tile_device.h, which also has
//   the larger tiles).
//   Global loads happen in A and stores in C; with k = 10 every access is a
//   64 B run of consecutive amplitudes, with S >= 6 a run of >= 512 B.
//
//   The phase layer exp(-i g C) (Sec. IV-B, Euler's formula) is applied to a
//   tile right after loading it in the first pass of a layer, and the
//   expectation sum C|psi|^2 (Sec. IV-D) is accumulated in the last pass, so
//   neither costs a sweep of its own.
//
//   Adjoint gradient (Sec. II-B, IV-C): with lam = C psi, a backward pass loads
//   (phi, lam), adds Im(conj(lam_z) phi_{z^2^j}) for every pair of the group
//   (this is Im <lam|X_j|phi>, unchanged by any mixer factor applied to both),
//   applies exp(+i b X_j) to both, and in the last pass of a layer adds
//   C Im(conj(lam) phi) and undoes the phase.  Layer states are recomputed by
//   these inverse layers; none is stored.  The "turn" pass fuses the last
//   forward group with the first backward group: it evolves psi through the
//   group, forms E and lam = C phi, then undoes the group on lam; phi after
//   the undo is exactly what memory already holds, so it is not written.
//
// Every reduction is a fixed-order tree (shuffle within a wave, then LDS),
// one partial per workgroup, summed by k_sum_slots in fixed order: results are
// bitwise reproducible.
#include "tile_device.h"

namespace qk {
namespace {

// ------------------------------------------------------------ reductions

// out[k] = scale * sum_{i < count} parts[k * stride + i], one workgroup per slot, fixed order.
__global__ __launch_bounds__(kThreads) void k_sum_slots(const double *parts, uint64_t count,
                                                        uint64_t stride, double scale, double *out)
{
    __shared__ double red[4];
    const double *p = parts + (uint64_t)blockIdx.x * stride;
    // eight loads in flight per thread (one by one: 430 us for 2^18 partials a slot, n = 30)
    double a[8] = {};
    for (uint64_t i = threadIdx.x; i < count; i += 8 * kThreads) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (i + r * kThreads < count) a[r] += p[i + r * kThreads];
    }
    const double acc = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) out[blockIdx.x] = scale * s;
}

// Gradient outputs in device memory from the summed slots (p <= 64 threads).
__global__ void k_gradient_out(const double *res, int p, double *E, double *dg, double *db)
{
    const int i = threadIdx.x;
    if (i == 0 && E) E[0] = res[0];
    if (i < p) {
        db[i] = 2.0 * res[1 + i];
        dg[i] = 2.0 * res[1 + p + i];
    }
}

// Expectation of a stored state: one partial per 4096 amplitudes.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_expect(const typename Tr<R>::V *psi,
                                                     const typename Tr<R>::CT *C, uint64_t N,
                                                     double *parts)
{
    __shared__ double red[4];
    const uint64_t b0 = (uint64_t)blockIdx.x * kTile;
    double acc = 0.0;
#pragma unroll 4
    for (int r = 0; r < kTile / kThreads; ++r) {
        const uint64_t z = b0 + (uint64_t)r * kThreads + threadIdx.x;
        if (z < N) acc += (double)C[z] * norm2(psi[z]);
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) parts[blockIdx.x] = s;
}

template <typename CT>
__global__ __launch_bounds__(kThreads) void k_minmax(const CT *C, uint64_t N, double *pmin,
                                                     double *pmax)
{
    __shared__ double red[2][kThreads];
    const uint64_t b0 = (uint64_t)blockIdx.x * kTile;
    double lo = INFINITY, hi = -INFINITY;
    for (int r = 0; r < kTile / kThreads; ++r) {
        const uint64_t z = b0 + (uint64_t)r * kThreads + threadIdx.x;
        if (z < N) {
            const double v = (double)C[z];
            lo = fmin(lo, v);
            hi = fmax(hi, v);
        }
    }
    red[0][threadIdx.x] = lo;
    red[1][threadIdx.x] = hi;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + w]);
            red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        pmin[blockIdx.x] = red[0][0];
        pmax[blockIdx.x] = red[1][0];
    }
}

__global__ __launch_bounds__(kThreads) void k_minmax_final(const double *pmin, const double *pmax,
                                                           uint64_t count, double *out)
{
    __shared__ double red[2][kThreads];
    double lo = INFINITY, hi = -INFINITY;
    for (uint64_t i = threadIdx.x; i < count; i += kThreads) {
        lo = fmin(lo, pmin[i]);
        hi = fmax(hi, pmax[i]);
    }
    red[0][threadIdx.x] = lo;
    red[1][threadIdx.x] = hi;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + w]);
            red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = red[0][0];
        out[1] = red[1][0];
    }
}

// ------------------------------------------------------------ cost diagonal

// A workgroup builds 4096 consecutive entries of the cost diagonal per
// iteration.  Thread (lane, wave) holds the 16 entries z = base | q << 6 |
// lane | wave << 10, q < 16, so every store of a wave is 64 consecutive
// entries, and z bits >= 10 are the same for the whole wavefront.  The terms
// arrive as pieces (cost_terms.cpp).  The workgroup brings kCostChunk of them
// into LDS with one coalesced read, each lane of a wavefront tests the wave-bit
// literals of one piece, and the wavefront then goes through the pieces that
// passed, in order: a lane adds the weight, or -0.0 if it fails the lane-bit
// literals (x + (-0.0) == x exactly in round-to-nearest, signed zeros included),
// to the entries q that the piece covers.  Each entry thus receives exactly
// the weights of its active terms, added one by one in the given term order, as
// the definition sums them.
// Small arrays are bound by the latency of reading the pieces: fetched one by
// one with scalar loads, each a miss in turn, they took 100 us at 2^21 entries
// and 230 pieces; this way it takes 27 us.
constexpr int kCostTileBits = 12;
constexpr int kCostChunk = 256;

template <typename CT>
__device__ __forceinline__ void store_costs(CT *__restrict__ C, uint64_t N, uint64_t zt, const double (&acc)[16])
{
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const uint64_t z = zt | ((uint64_t)q << 6);
        if (z < N) C[z] = (CT)acc[q];
    }
}

// acc[q] += w in the lanes of `in`, for the entries q of qpat (all lanes are
// active here).  The sums stay in their registers and the execution mask says
// who adds: written in C++, the same choice costs copies of all 16 sums for each
// term (47 us instead of 27 where the comment above counts).  The scalar
// instructions ahead of the first addition are also the wait states that it
// needs after the lane reads that made w.
__device__ __forceinline__ void add_covered(double (&acc)[16], double w, uint64_t in, uint32_t qpat)
{
    uint64_t all;
#define QK_ADD(q) "v_add_f64 %[a" #q "], %[a" #q "], %[w]\n\t"
#define QK_ADD_IF(q) "s_bitcmp1_b32 %[p], " #q "\n\ts_cselect_b64 exec, %[in], 0\n\t" QK_ADD(q)
#define QK_ALL(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
    asm("s_mov_b64 %[all], exec\n\t"
        "s_cmpk_eq_u32 %[p], 0xffff\n\t"
        "s_cbranch_scc1 1f\n\t" QK_ALL(QK_ADD_IF)
        "s_branch 2f\n"
        "1:\n\t"
        "s_mov_b64 exec, %[in]\n\t" QK_ALL(QK_ADD)
        "2:\n\t"
        "s_mov_b64 exec, %[all]"
        : [all] "=&s"(all), [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]),
          [a4] "+v"(acc[4]), [a5] "+v"(acc[5]), [a6] "+v"(acc[6]), [a7] "+v"(acc[7]), [a8] "+v"(acc[8]),
          [a9] "+v"(acc[9]), [a10] "+v"(acc[10]), [a11] "+v"(acc[11]), [a12] "+v"(acc[12]),
          [a13] "+v"(acc[13]), [a14] "+v"(acc[14]), [a15] "+v"(acc[15])
        : [w] "s"(w), [in] "s"(in), [p] "s"(qpat)
        : "scc");
#undef QK_ALL
#undef QK_ADD_IF
#undef QK_ADD
}

template <typename CT>
__global__ __launch_bounds__(kThreads) void k_cost_pieces(CT *__restrict__ C, uint64_t N,
                                                          const CostPiece *__restrict__ P,
                                                          int64_t count, double offset)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int kWords = sizeof(CostPiece) / 8;
    __shared__ CostPiece pieces[kCostChunk];
    for (uint64_t tile = blockIdx.x; (tile << kCostTileBits) < N; tile += gridDim.x) {
        const uint64_t zw = (tile << kCostTileBits) | ((uint64_t)wave << 10);
        double acc[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = offset;
        for (int64_t k0 = 0; k0 < count; k0 += kCostChunk) {
            const int here = (int)(count - k0 < kCostChunk ? count - k0 : kCostChunk);
            uint64_t word[kCostChunk * kWords / kThreads];  // all loads in flight at once
#pragma unroll
            for (int i = 0; i < kCostChunk * kWords / kThreads; ++i) {
                const int x = i * kThreads + (int)threadIdx.x;
                __builtin_memcpy(&word[i], (const char *)(P + k0) + 8 * (x < here * kWords ? x : 0), 8);
            }
            __syncthreads();  // the chunk before is done with
#pragma unroll
            for (int i = 0; i < kCostChunk * kWords / kThreads; ++i)
                __builtin_memcpy((char *)pieces + 8 * (i * kThreads + (int)threadIdx.x), &word[i], 8);
            __syncthreads();
            for (int g = 0; g < here; g += 64) {
                const CostPiece &pc = pieces[g + (int)lane < here ? g + (int)lane : here - 1];
                const uint64_t wb = (uint64_t)__double_as_longlong(pc.wq.w);
                const uint32_t wlo = (uint32_t)wb, whi = (uint32_t)(wb >> 32), qp = pc.wq.qpat, ln = pc.lanes;
                uint64_t todo = __ballot(g + (int)lane < here && (zw & pc.umask) == pc.uval);
                while (todo) {
                    const int b = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    const uint32_t l = __builtin_amdgcn_readlane(ln, b);
                    const uint32_t qpat = __builtin_amdgcn_readlane(qp, b);
                    const double w = __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane(whi, b) << 32 |
                                                                      (uint32_t)__builtin_amdgcn_readlane(wlo, b)));
                    add_covered(acc, w, __ballot((lane & l & 63u) == (l >> 8)), qpat);
                }
            }
        }
        store_costs(C, N, zw | lane, acc);
    }
}

template <typename R>
__global__ __launch_bounds__(kThreads) void k_fill_plus(typename Tr<R>::V *psi, uint64_t N, R amp)
{
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t z = (uint64_t)blockIdx.x * kThreads + threadIdx.x; z < N; z += stride) {
        typename Tr<R>::V v;
        v.x = amp;
        v.y = (R)0;
        psi[z] = v;
    }
}

__global__ __launch_bounds__(kThreads) void k_widen(const float *C32, double *out, uint64_t N)
{
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t z = (uint64_t)blockIdx.x * kThreads + threadIdx.x; z < N; z += stride)
        out[z] = (double)C32[z];
}

// out[z] = out[2 half - 1 - z] = in[z]: a whole array from the half of a folded
// one (z and ~z hold the same value).  Bound by memory: the half is read once,
// where copying an unfolded array would read it all.
// W is the unit of the copy: the entry, or a part of it that the output's
// alignment allows (`words` of them make an entry).
template <typename W>
__global__ __launch_bounds__(kThreads) void k_unfold_words(const W *in, uint64_t half, uint32_t words, W *out)
{
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < half * words; i += stride) {
        const W v = in[i];
        out[i] = v;
        out[(2 * half - 1 - i / words) * words + i % words] = v;
    }
}
// x[i] <-> x[count - 1 - i]
template <typename W>
__global__ __launch_bounds__(kThreads) void k_reverse(W *x, uint64_t count)
{
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < count / 2; i += stride) {
        const W a = x[i], b = x[count - 1 - i];
        x[i] = b;
        x[count - 1 - i] = a;
    }
}
// The same as k_unfold_words for cost entries, fp32 widened to fp64.
__global__ __launch_bounds__(kThreads) void k_unfold_widen(const float *in, uint64_t half, double *out)
{
    const uint64_t stride = (uint64_t)gridDim.x * kThreads;
    for (uint64_t z = (uint64_t)blockIdx.x * kThreads + threadIdx.x; z < half; z += stride) {
        const double v = (double)in[z];
        out[z] = v;
        out[2 * half - 1 - z] = v;
    }
}

// ------------------------------------------------------------ sampling

// Stored index of z: a folded state keeps z >= N/2 at its complement.
__device__ __forceinline__ uint64_t stored(uint64_t z, uint64_t N, bool folded)
{
    return folded && z >= (N >> 1) ? N - 1 - z : z;
}

// Philox-4x32-10 (Salmon et al., SC'11): ten rounds of the two 32x32->64
// multiplies with M0 = 0xD2511F53 and M1 = 0xCD9E8D57, key bumped by the Weyl
// constants 0x9E3779B9 / 0xBB67AE85 between rounds.
__device__ __forceinline__ double philox_uniform53(uint64_t seed, uint64_t s)
{
    uint32_t x0 = (uint32_t)s, x1 = (uint32_t)(s >> 32), x2 = 0u, x3 = 0u;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = 0xD2511F53u * x0, hi0 = __umulhi(0xD2511F53u, x0);
        const uint32_t lo1 = 0xCD9E8D57u * x2, hi1 = __umulhi(0xCD9E8D57u, x2);
        const uint32_t y0 = hi1 ^ x1 ^ k0, y2 = hi0 ^ x3 ^ k1;
        x0 = y0;
        x1 = lo1;
        x2 = y2;
        x3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    const uint64_t w = ((uint64_t)x1 << 32) | x0;
    return (double)(w >> 11) * 0x1.0p-53;
}

// Mass of each sub-block of 2^sbits amplitudes (sbits != 8): one wave per
// sub-block, each lane sums a fixed set of elements in order, then a shuffle tree.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_submass(const typename Tr<R>::V *psi, uint64_t N,
                                                      bool folded, int sbits, uint64_t nsub, double *sub)
{
    const uint64_t j = (uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    if (j >= nsub) return;  // whole wave exits together
    const uint64_t sb = 1ull << sbits, z0 = j << sbits;
    double acc = 0.0;
    for (uint64_t i = lane; i < sb; i += 64) {
        const uint64_t z = z0 + i;
        if (z < N) acc += norm2(psi[stored(z, N, folded)]);
    }
    acc = wave_sum(acc);
    if (lane == 0) sub[j] = acc;
}

// x of another lane of the row of 16 (DPP control CTRL).
template <int CTRL>
__device__ __forceinline__ double row_lane(double x)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, true));
}
// wave_sum (the same pairs in the same order) without LDS: halves and rows by lane
// swaps; after the pairs 8 apart agree, a rotation by 4 reaches the pairs 4 apart.
__device__ __forceinline__ double wave_sum_lanes(double x)
{
    {
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
        x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
        x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    x += row_lane<0x128>(x);
    x += row_lane<0x124>(x);
    x += row_lane<0x4E>(x);
    return x + row_lane<0xB1>(x);
}

// The same for sub-blocks of 256 amplitudes (n in 8..32), of which `count` are
// stored.  The mirror image of a folded state's sub-block holds the same elements,
// lanes and order reversed: its sum is taken from the same read (the tree over
// reversed lanes pairs the same sums).  With `fine`, also the masses of the
// sub-block's 16 runs of 16 amplitudes, in any order of summing (k_shots).
// Bound by memory: the 1 GiB of n = 26 take 165 us, 190 with `fine`, whose 32 MiB
// are kept for the shots (two and four sub-blocks per wave: 201 and 207).
template <typename R>
__global__ __launch_bounds__(kThreads) void k_submass256(const typename Tr<R>::V *psi, uint64_t count, bool folded,
                                                         uint64_t nsub, double *sub, double *fine)
{
    const uint64_t j = (uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    if (j >= count) return;  // whole wave exits together
    double q[4], a = 0.0, b = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) q[r] = norm2(psi[(j << 8) + lane + 64 * r]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        a += q[r];
        b += q[3 - r];
    }
    a = wave_sum_lanes(a);
    if (folded) b = wave_sum_lanes(b);
    if (lane == 0) {
        sub[j] = a;
        if (folded) sub[nsub - 1 - j] = b;
    }
    if (fine) {
        double f = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double x = q[r];
            x += row_lane<0xB1>(x);
            x += row_lane<0x4E>(x);
            x += row_lane<0x141>(x);
            x += row_lane<0x140>(x);
            f = (lane & 15u) == (uint32_t)r ? x : f;
        }
        if ((lane & 15u) < 4) fine[j * 16 + (lane & 15u) * 4 + (lane >> 4)] = f;
    }
}

constexpr int kScanChunk = kThreads * 16;  // entries per workgroup in the scan

// Per-chunk totals.
__global__ __launch_bounds__(kThreads) void k_scan_partial(const double *in, uint64_t count,
                                                           double *tot)
{
    __shared__ double red[4];
    const uint64_t c0 = (uint64_t)blockIdx.x * kScanChunk;
    double acc = 0.0;
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = c0 + (uint64_t)threadIdx.x * 16 + r;
        if (i < count) acc += in[i];
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) tot[blockIdx.x] = s;
}

// Exclusive scan of `x` across the 256 threads of a block (thread-ordered);
// returns the exclusive prefix for this thread and the block total in *total.
__device__ __forceinline__ double block_exclusive(double x, double *sh, double *total)
{
    sh[threadIdx.x] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        // a chain of 256 adds; the reads of 16 of them at a time do not wait for it
        // (one by one the chain took 6 of the kernel's 8 us)
        double run = 0.0;
        for (int i = 0; i < kThreads; i += 16) {
            double v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = sh[i + r];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                sh[i + r] = run;
                run += v[r];
            }
        }
        sh[kThreads] = run;
    }
    __syncthreads();
    const double r = sh[threadIdx.x];
    *total = sh[kThreads];
    __syncthreads();
    return r;
}

// Exclusive scan of the chunk totals (at most kScanChunk of them) in place;
// tot[nchunks] receives the grand total.
__global__ __launch_bounds__(kThreads) void k_scan_top(double *tot, uint64_t nchunks)
{
    __shared__ double sh[kThreads + 1];
    double v[16];
    double local = 0.0;
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = (uint64_t)threadIdx.x * 16 + r;
        v[r] = i < nchunks ? tot[i] : 0.0;
        local += v[r];
    }
    double total;
    double run = block_exclusive(local, sh, &total);
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = (uint64_t)threadIdx.x * 16 + r;
        if (i < nchunks) tot[i] = run;
        run += v[r];
    }
    if (threadIdx.x == 0) tot[nchunks] = total;
}

// out[i] = sum_{k < i} in[k] for i <= count (out[count] = *total_out = total).
__global__ __launch_bounds__(kThreads) void k_scan_final(const double *in, uint64_t count,
                                                         const double *tot, uint64_t nchunks,
                                                         double *out, double *total_out)
{
    __shared__ double sh[kThreads + 1];
    const uint64_t c0 = (uint64_t)blockIdx.x * kScanChunk;
    double v[16];
    double local = 0.0;
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = c0 + (uint64_t)threadIdx.x * 16 + r;
        v[r] = i < count ? in[i] : 0.0;
        local += v[r];
    }
    double total;
    double run = tot[blockIdx.x] + block_exclusive(local, sh, &total);
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = c0 + (uint64_t)threadIdx.x * 16 + r;
        if (i < count) out[i] = run;
        run += v[r];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        out[count] = tot[nchunks];
        *total_out = tot[nchunks];
    }
}

// What lanes of a wave wrote to LDS before it, the others read after it, and the
// other way round.
__device__ __forceinline__ void wave_exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// W shots per wave (grid-stride), a lane each: u -> target t = u * total, binary search
// over the sub-block prefix, then a sequential scan inside the sub-block for the first
// z whose cumulative mass exceeds t.  A zero-probability z never satisfies the
// test (its cumulative mass equals its predecessor's), so it is never returned.
//
// The 64 scans of a wave are in 64 different sub-blocks.  Read by its own lane, each
// amplitude costs a cache line (1.20 ms for 10^6 shots at n = 26, complex128, also
// with 16 loads ahead of the chain of sums).  Here eight lanes read eight consecutive
// amplitudes of one shot, and the masses go to the shot's lane through LDS: 0.43 ms,
// of which 0.18 are the chains (n = 14) and the rest 2.1 GB of reads.
//
// With `fine`, the masses of the runs of 16 amplitudes, a shot needs 128 bytes of
// those and the 16 amplitudes of one run: 0.12 ms instead of 0.45 (1024 shots at n =
// 22: 11.5 instead of 28 us).  The sums then round
// otherwise, by less than 2^-44 T in all (256 additions against 32, each off by at
// most 2^-53 of a sum of at most T): the z found is that of the scan unless one of
// the two sums around t is within 2^-43 T of it, in which case the shot is scanned.
template <typename R, int W>
__global__ __launch_bounds__(kThreads) void k_shots(const typename Tr<R>::V *psi,
                                                    const typename Tr<R>::CT *C, uint64_t N,
                                                    bool folded, int sbits, const double *pre, uint64_t nsub,
                                                    const double *fine, int64_t shots, uint64_t seed, uint64_t *zout,
                                                    double *cout)
{
    constexpr int kLoads = 8, kRows = W / 8, kStep = 8 * kLoads / kRows;  // loads in flight; amplitudes per turn
    __shared__ double mass[kThreads / 64][W][kStep + 1];
    const double T = pre[nsub];
    if (!(T > 0.0) || T == INFINITY) return;  // no shots from such a state (the caller reports it)
    const uint32_t lane = threadIdx.x & 63u, sub = lane & 7u, row = lane >> 3;
    double (*m)[kStep + 1] = mass[threadIdx.x >> 6];
    const uint64_t sb = 1ull << sbits;
    const uint64_t stride = (uint64_t)gridDim.x * (kThreads / 64) * W;
    const uint64_t first = ((uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)) * W;
    for (uint64_t s0 = first; s0 < (uint64_t)shots; s0 += stride) {
        const uint64_t s = s0 + lane;
        const bool mine = lane < W && s < (uint64_t)shots;
        const double t = philox_uniform53(seed, s) * T;
        uint64_t lo = 0, hi = mine ? nsub - 1 : 0;  // smallest j with pre[j+1] > t
        while (lo < hi) {
            const uint64_t mid = lo + (hi - lo) / 2;
            if (pre[mid + 1] > t) hi = mid;
            else lo = mid + 1;
        }
        // the shots whose amplitudes this lane reads: row, row + 8, ..
        uint64_t zr[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) zr[k] = (uint64_t)__shfl((long long)lo, k * 8 + row) << sbits;
        const uint64_t z0 = lo << sbits;
        // acc never decreases: the amplitudes with acc <= t are the ones before z
        double acc = pre[lo];
        uint32_t before = 0;
        bool found = !mine;
        if (fine) {
#pragma unroll
            for (int k = 0; k < kRows; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    m[k * 8 + row][8 * i + sub] = fine[stored((zr[k] >> 4) + 8 * i + sub, N >> 4, folded)];
            wave_exchange();
            double under = acc;  // the sum before the run, then before the amplitude
            uint32_t run = 0;
            if (!found) {
                double sum = acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    sum += m[lane][r];
                    if (sum <= t) under = sum;
                    run += sum <= t ? 1u : 0u;
                }
            }
            wave_exchange();
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const uint64_t zb = zr[k] + 16 * min((uint32_t)__shfl((int)run, k * 8 + row), 15u);
#pragma unroll
                for (int i = 0; i < 2; ++i) m[k * 8 + row][8 * i + sub] = norm2(psi[stored(zb + 8 * i + sub, N, folded)]);
            }
            wave_exchange();
            if (!found) {
                double sum = under, over = t;
                uint32_t in = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    sum += m[lane][r];
                    if (sum <= t) under = sum;
                    else if (in == (uint32_t)r) over = sum;
                    in += sum <= t ? 1u : 0u;
                }
                const double eps = T * 0x1p-43;
                found = run < 16 && in < 16 && over > t + eps && under < t - eps;
                before = found ? 16 * run + in : 0u;
            }
            wave_exchange();
        }
        for (uint64_t d = 0; d < sb; d += kStep) {
            const uint64_t open = __ballot(!found);
            if (!open) break;
            typename Tr<R>::V v[kLoads];
#pragma unroll
            for (int k = 0; k < kLoads; ++k)
                if ((open >> ((k % kRows) * 8 + row)) & 1ull)
                    v[k] = psi[stored(zr[k % kRows] + min(d + (k / kRows) * 8 + sub, sb - 1), N, folded)];
#pragma unroll
            for (int k = 0; k < kLoads; ++k) {
                const uint32_t e = (k / kRows) * 8 + sub;
                if ((open >> ((k % kRows) * 8 + row)) & 1ull)
                    m[(k % kRows) * 8 + row][e] = d + e < sb ? norm2(v[k]) : 0.0;
            }
            wave_exchange();
            if (!found) {
#pragma unroll
                for (int r = 0; r < kStep; ++r) {
                    acc += m[lane][r];
                    before += acc > t ? 0u : 1u;
                }
                found = acc > t;
            }
            wave_exchange();
        }
        uint64_t zsel = z0 + before;
        if (!found) {
            // rounding left t at the sub-block's end: its last amplitude that is not zero
            for (zsel = z0 + sb - 1; zsel > z0 && !(norm2(psi[stored(zsel, N, folded)]) > 0.0);) --zsel;
        }
        if (mine) {
            zout[s] = zsel;
            if (cout) cout[s] = (double)C[stored(zsel, N, folded)];
        }
    }
}

// Workgroups of a cost-diagonal launch: one per 4096 entries, at most 2^20.
inline unsigned cost_grid(uint64_t N)
{
    const uint64_t t = (N + (1ull << kCostTileBits) - 1) >> kCostTileBits;
    return (unsigned)(t < (1ull << 20) ? t : (1ull << 20));
}

inline unsigned grid_for(uint64_t N, uint64_t cap = 1ull << 20)
{
    uint64_t g = (N + kThreads - 1) / kThreads;
    if (g > cap) g = cap;
    if (g == 0) g = 1;
    return (unsigned)g;
}

}  // namespace

// ------------------------------------------------------------ launchers

int static_spectators(const Geometry &g, int TB, int mode)
{
    const uint32_t t = g.tmask;
    if ((int)g.tbits != TB || t == 0) return -1;
    const int S = __builtin_ctz(t);
    if (t != (((1u << TB) - 1u) & ~((1u << S) - 1u))) return -1;  // not "every bit from S up"
    if (S == 0) return 0;
    return (S >= 2 && S <= 7 && mode != kTurnPhase) ? S : -1;
}

// A pass with a spectator class that has its own kernels (every full-tile pass
// whose S lowest tile bits are spectators, S = 0 or 2..7) runs them;
// any other pass runs the kernels that read the target mask at run time.
hipError_t launch_pass(int mode, bool c64, const PassArgs &a, uint64_t nblocks, hipStream_t s)
{
    int sp = static_spectators(a.geo, tile_bits(c64), mode);
    // a class's kernels fix whether their accesses stream, and take every phase
    // argument in the fast reduction's range
    if (sp >= 0 && stream_class(sp) != ((a.flags & kStream) != 0)) sp = -1;
    if (a.flags & kFarPhase) sp = -1;
    if (!c64) {
        switch (sp) {
        case 0: return launch_pass_sp<double, 0>(mode, a, nblocks, s);
        case 2: return launch_pass_sp<double, 2>(mode, a, nblocks, s);
        case 3: return launch_pass_sp<double, 3>(mode, a, nblocks, s);
        case 4: return launch_pass_sp<double, 4>(mode, a, nblocks, s);
        case 5: return launch_pass_sp<double, 5>(mode, a, nblocks, s);
        case 6: return launch_pass_sp<double, 6>(mode, a, nblocks, s);
        case 7: return launch_pass_sp<double, 7>(mode, a, nblocks, s);
        default: return launch_pass_sp<double, -1>(mode, a, nblocks, s);
        }
    }
    switch (sp) {
    case 0: return launch_pass_sp<float, 0>(mode, a, nblocks, s);
    case 2: return launch_pass_sp<float, 2>(mode, a, nblocks, s);
    case 3: return launch_pass_sp<float, 3>(mode, a, nblocks, s);
    case 4: return launch_pass_sp<float, 4>(mode, a, nblocks, s);
    case 5: return launch_pass_sp<float, 5>(mode, a, nblocks, s);
    case 6: return launch_pass_sp<float, 6>(mode, a, nblocks, s);
    case 7: return launch_pass_sp<float, 7>(mode, a, nblocks, s);
    default: return launch_pass_sp<float, -1>(mode, a, nblocks, s);
    }
}

hipError_t launch_quad(int mode, bool c64, int tbits, const PassArgs &a, uint64_t nblocks, hipStream_t s)
{
    return c64 ? launch_quad_real<float>(mode, tbits, a, nblocks, s) : launch_quad_real<double>(mode, tbits, a, nblocks, s);
}

hipError_t launch_many(int mode, const PassArgs &a, const ManyArgs &m, uint64_t nblocks, unsigned count,
                       hipStream_t s)
{
    int sp = static_spectators(a.geo, kTileBits, mode);
    if (sp >= 0 && stream_class(sp) != ((a.flags & kStream) != 0)) sp = -1;
    switch (sp) {
    case 0: return launch_many_sp<0>(mode, a, m, nblocks, count, s);
    case 2: return launch_many_sp<2>(mode, a, m, nblocks, count, s);
    case 3: return launch_many_sp<3>(mode, a, m, nblocks, count, s);
    case 4: return launch_many_sp<4>(mode, a, m, nblocks, count, s);
    case 5: return launch_many_sp<5>(mode, a, m, nblocks, count, s);
    case 6: return launch_many_sp<6>(mode, a, m, nblocks, count, s);
    case 7: return launch_many_sp<7>(mode, a, m, nblocks, count, s);
    default: return launch_many_sp<-1>(mode, a, m, nblocks, count, s);
    }
}

hipError_t launch_large(int mode, bool c64, const PassArgs &a, uint64_t nblocks, hipStream_t s)
{
    const int sp = static_spectators(a.geo, tile_bits(c64) + 1, mode);
    if (sp < 0 || stream_class(sp) != ((a.flags & kStream) != 0) || (a.flags & kFarPhase)) return hipErrorInvalidValue;
    if (!c64) {
        switch (sp) {
        case 0: return launch_large_sp<double, 0>(mode, a, nblocks, s);
        case 2: return launch_large_sp<double, 2>(mode, a, nblocks, s);
        case 3: return launch_large_sp<double, 3>(mode, a, nblocks, s);
        }
        return hipErrorInvalidValue;
    }
    switch (sp) {
    case 0: return launch_large_sp<float, 0>(mode, a, nblocks, s);
    case 3: return launch_large_sp<float, 3>(mode, a, nblocks, s);
    case 4: return launch_large_sp<float, 4>(mode, a, nblocks, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_sum_slots(const double *parts, uint64_t count, uint64_t stride, int nslots, double scale,
                            double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_slots, dim3(nslots), dim3(kThreads), 0, s, parts, count, stride, scale, out);
    return hipGetLastError();
}

hipError_t launch_gradient_out(const double *res, int p, double *E, double *dgamma, double *dbeta,
                               hipStream_t s)
{
    if (p > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gradient_out, dim3(1), dim3(64), 0, s, res, p, E, dgamma, dbeta);
    return hipGetLastError();
}

hipError_t launch_cost_pieces(bool c64, void *C, int n, const CostPiece *pieces, int64_t count,
                              double offset, hipStream_t s)
{
    const uint64_t N = 1ull << n;
    if (c64)
        hipLaunchKernelGGL(k_cost_pieces<float>, dim3(cost_grid(N)), dim3(kThreads), 0, s,
                           (float *)C, N, pieces, count, offset);
    else
        hipLaunchKernelGGL(k_cost_pieces<double>, dim3(cost_grid(N)), dim3(kThreads), 0, s,
                           (double *)C, N, pieces, count, offset);
    return hipGetLastError();
}

hipError_t launch_fill_plus(bool c64, void *psi, int n, uint64_t count, hipStream_t s)
{
    const double amp = 1.0 / sqrt((double)(1ull << n));
    if (c64)
        hipLaunchKernelGGL(k_fill_plus<float>, dim3(grid_for(count)), dim3(kThreads), 0, s,
                           (Tr<float>::V *)psi, count, (float)amp);
    else
        hipLaunchKernelGGL(k_fill_plus<double>, dim3(grid_for(count)), dim3(kThreads), 0, s,
                           (Tr<double>::V *)psi, count, amp);
    return hipGetLastError();
}

hipError_t launch_unfold(const void *in, uint64_t half, int entry_bytes, void *out, hipStream_t s)
{
    const uintptr_t a = (uintptr_t)out;
    const auto go = [&](auto w) {
        using W = decltype(w);
        const uint32_t words = (uint32_t)(entry_bytes / sizeof(W));
        hipLaunchKernelGGL(k_unfold_words<W>, dim3(grid_for(half * words)), dim3(kThreads), 0, s, (const W *)in, half,
                           words, (W *)out);
        return hipGetLastError();
    };
    if (entry_bytes == 16 && a % 16 == 0) return go(uint4{});
    if (entry_bytes >= 8 && a % 8 == 0) return go(uint64_t{});
    return a % 4 == 0 ? go(uint32_t{}) : go(uint8_t{});
}

hipError_t launch_reverse(void *x, uint64_t count, int entry_bytes, hipStream_t s)
{
    const dim3 grid(grid_for(count / 2)), block(kThreads);
    if (entry_bytes == 16) hipLaunchKernelGGL(k_reverse<uint4>, grid, block, 0, s, (uint4 *)x, count);
    else if (entry_bytes == 8) hipLaunchKernelGGL(k_reverse<uint64_t>, grid, block, 0, s, (uint64_t *)x, count);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_unfold_widen(const float *in, uint64_t half, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_unfold_widen, dim3(grid_for(half)), dim3(kThreads), 0, s, in, half, out);
    return hipGetLastError();
}

hipError_t launch_expect(bool c64, const void *psi, const void *C, int n, double *parts,
                         hipStream_t s)
{
    const uint64_t N = 1ull << n;
    const unsigned nb = (unsigned)((N + kTile - 1) / kTile);
    if (c64)
        hipLaunchKernelGGL(k_expect<float>, dim3(nb), dim3(kThreads), 0, s, (const Tr<float>::V *)psi,
                           (const float *)C, N, parts);
    else
        hipLaunchKernelGGL(k_expect<double>, dim3(nb), dim3(kThreads), 0, s,
                           (const Tr<double>::V *)psi, (const double *)C, N, parts);
    return hipGetLastError();
}

hipError_t launch_minmax(bool c64, const void *C, int n, double *pmin, double *pmax,
                         hipStream_t s)
{
    const uint64_t N = 1ull << n;
    const unsigned nb = (unsigned)((N + kTile - 1) / kTile);
    if (c64)
        hipLaunchKernelGGL(k_minmax<float>, dim3(nb), dim3(kThreads), 0, s, (const float *)C, N,
                           pmin, pmax);
    else
        hipLaunchKernelGGL(k_minmax<double>, dim3(nb), dim3(kThreads), 0, s, (const double *)C,
                           N, pmin, pmax);
    return hipGetLastError();
}

hipError_t launch_minmax_final(const double *pmin, const double *pmax, uint64_t count,
                               double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_minmax_final, dim3(1), dim3(kThreads), 0, s, pmin, pmax, count, out);
    return hipGetLastError();
}

hipError_t launch_widen_cost(const float *C32, double *out, uint64_t N, hipStream_t s)
{
    hipLaunchKernelGGL(k_widen, dim3(grid_for(N)), dim3(kThreads), 0, s, C32, out, N);
    return hipGetLastError();
}

int sample_subblock_bits(int n)
{
    int sb = n - 24 > 8 ? n - 24 : 8;
    return sb < n ? sb : n;
}

uint64_t scan_scratch_doubles(uint64_t count)
{
    return (count + kScanChunk - 1) / kScanChunk + 1;
}

// The runs' masses save the shots' reads and a chain of up to 256 sums, and cost
// the writing of 8 bytes for 16 amplitudes: up to 2^25 stored amplitudes they pay for
// any number of shots (whole call, us, without and with: n = 14 36 and 30, 22 57 and
// 44, 24 84 and 72), at 2^26 from 2^16 shots on (1024 shots 221 and 228, 64 000 254
// and 232), beyond from as many more.  Up to 128 MiB of them are kept.
uint64_t sample_fine_doubles(int n, bool folded, int64_t shots)
{
    const uint64_t held = 1ull << (folded ? n - 1 : n);
    return sample_subblock_bits(n) == 8 && n <= 28 && (held <= 1ull << 25 || (uint64_t)shots >= held >> 10)
               ? held >> 4
               : 0;
}

hipError_t launch_submass(bool c64, const void *psi, int n, bool folded, int sbits, double *sub, double *fine,
                          hipStream_t s)
{
    const uint64_t N = 1ull << n, nsub = 1ull << (n - sbits);
    if (sbits == 8) {
        const uint64_t count = folded ? nsub / 2 : nsub;
        const dim3 grid((unsigned)((count + 3) / 4));
        if (c64)
            hipLaunchKernelGGL(k_submass256<float>, grid, dim3(kThreads), 0, s, (const Tr<float>::V *)psi, count,
                               folded, nsub, sub, fine);
        else
            hipLaunchKernelGGL(k_submass256<double>, grid, dim3(kThreads), 0, s, (const Tr<double>::V *)psi, count,
                               folded, nsub, sub, fine);
        return hipGetLastError();
    }
    const unsigned nb = (unsigned)((nsub + 3) / 4);
    if (c64)
        hipLaunchKernelGGL(k_submass<float>, dim3(nb), dim3(kThreads), 0, s, (const Tr<float>::V *)psi,
                           N, folded, sbits, nsub, sub);
    else
        hipLaunchKernelGGL(k_submass<double>, dim3(nb), dim3(kThreads), 0, s,
                           (const Tr<double>::V *)psi, N, folded, sbits, nsub, sub);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan(const double *in, uint64_t count, double *out, double *scratch,
                                 double *total, hipStream_t s)
{
    const uint64_t nchunks = (count + kScanChunk - 1) / kScanChunk;
    if (nchunks > (uint64_t)kScanChunk) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_scan_partial, dim3((unsigned)nchunks), dim3(kThreads), 0, s, in, count,
                       scratch);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kThreads), 0, s, scratch, nchunks);
    hipLaunchKernelGGL(k_scan_final, dim3((unsigned)nchunks), dim3(kThreads), 0, s, in, count,
                       scratch, nchunks, out, total);
    return hipGetLastError();
}

hipError_t launch_shots(bool c64, const void *psi, const void *C, int n, bool folded, int sbits,
                        const double *pre, uint64_t nsub, const double *fine, int64_t shots, uint64_t seed,
                        uint64_t *z, double *cost, hipStream_t s)
{
    const uint64_t N = 1ull << n;
    // 8 shots a wave, whose sub-blocks are read 64 amplitudes at a time, while that
    // gives every SIMD a wave or few; 32 a wave, whose chains of sums fill four times
    // the lanes, beyond (n = 20, both in us: 16 000 shots 64 and 87, 64 000 89 and 93,
    // 250 000 164 and 142, 10^6 473 and 327).  With the runs' masses a shot has little
    // to read, and the lanes count from 2^14 shots on (n = 22, us per call: 1024 shots
    // 42 and 45, 16 000 44 and 44, 64 000 53 and 45).
#define QK_SHOTS(R, W)                                                                                         \
    hipLaunchKernelGGL((k_shots<R, W>), dim3(grid_for((uint64_t)shots * (64 / W))), dim3(kThreads), 0, s,          \
                       (const Tr<R>::V *)psi, (const Tr<R>::CT *)C, N, folded, sbits, pre, nsub, fine, shots, seed, z, cost)
    if (shots <= (fine ? 1 << 14 : 1 << 16)) {
        if (c64) QK_SHOTS(float, 8);
        else QK_SHOTS(double, 8);
    } else {
        if (c64) QK_SHOTS(float, 32);
        else QK_SHOTS(double, 32);
    }
#undef QK_SHOTS
    return hipGetLastError();
}

}  // namespace qk
