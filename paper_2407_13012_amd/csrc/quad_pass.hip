// Pass kernels of states that do not fill the card (quad_tile_bits): the
// passes of passes.hip on tiles of 2^M amplitudes, M = 10, 11 or 12, with four
// amplitudes per thread (quad.h).
//
// A sweep of such a state is bound by the time of one workgroup: with 4096
// amplitudes in 256 threads an n = 17 MaxCut state was 16 workgroups of 14-19 us
// on 256 CUs.  Tiles of 1024 amplitudes make 64 of them with a quarter of the
// work each; the tile grows with n as far as two sweeps per layer need it.
// E + G at p = 6, complex128 MaxCut: n = 17 230 -> 102 us (a sweep 14-19 -> 5-8 us).
//
// Compiled once per QK_QUAD_REAL (double or float).
#include "many_device.h"
#include "quad.h"

#ifndef QK_QUAD_REAL
#error "QK_QUAD_REAL (double or float) must be defined"
#endif
#ifndef QK_PASS_MANY  // 1 in the complex128 unit: with the sweeps of the batched engine
#define QK_PASS_MANY 0
#endif

namespace qk {
namespace {

template <typename R, int M>
struct QuadLds {
    typename Tr<R>::V b0[1 << M], b1[1 << M];
    double red[4 * ((1 << M) / 256)];
};

// The other arrangement.
template <int M, typename R>
__device__ __forceinline__ void turn_to(One<R> &s, Place &w, QuadLds<R, M> &m, uint32_t tid)
{
    lds_barrier();
    put<M>(s.f, m.b0, w, tid);
    lds_barrier();
    w = Place{w.arr ^ 1, 0};
    get<M>(s.f, m.b0, w, tid, 0u);
}
template <int M, typename R>
__device__ __forceinline__ void turn_to(Two<R> &s, Place &w, QuadLds<R, M> &m, uint32_t tid)
{
    lds_barrier();
    put<M>(s.f, m.b0, w, tid);
    put<M>(s.l, m.b1, w, tid);
    lds_barrier();
    w = Place{w.arr ^ 1, 0};
    get<M>(s.f, m.b0, w, tid, 0u);
    get<M>(s.l, m.b1, w, tid, 0u);
}

template <typename R, int M, int MODE, bool TM, bool TM2>
__device__ __forceinline__ void quad_body(const PassArgs &a, QuadLds<R, M> &m)
{
    using V = typename Tr<R>::V;
    using CT = typename Tr<R>::CT;
    constexpr int NW = (1 << M) / 256;
    constexpr bool kOne = MODE == kFwd || MODE == kFwdFuse, kFuse = MODE == kFwdFuse || MODE == kBwdFuse;
    const uint32_t tid = threadIdx.x, b = blockIdx.x;
    const Geometry &g = a.geo;
    const uint64_t base = tile_base(xcd_tile(b, a.xcd_g), g);
    const uint32_t mask = g.tmask;
    V *psi = (V *)a.psi;
    V *lam = (V *)a.lam;
    const CT *cost = (const CT *)a.cost;
    // places a thread's amplitudes pass through: loaded in A; in B before and after
    // its rotations (entry, mid); back in A
    const Place wl{0, 0}, wm{1, M >= 11 ? 1 : 0}, we{0, 1};
    auto at = [&](Place w, uint32_t r) { return base ^ dep(elem_at<M>(w, tid, r), g); };
    const bool phaseIn = MODE == kFwd && (a.flags & kPhaseIn);
    const bool wantE = MODE == kTurn || (MODE == kFwd && (a.flags & kEOut));
    const bool phaseOut = MODE == kBwdFuse || (MODE == kBwd && (a.flags & kPhaseOut));
    double accE = 0.0, accG = 0.0, accB2 = 0.0;
    CT cin[4], cv[4];
    if (phaseIn) {
#pragma unroll
        for (int r = 0; r < 4; ++r) cin[r] = cost[at(wl, r)];
    }
    if (wantE || phaseOut || MODE == kFwdFuse) {
#pragma unroll
        for (int r = 0; r < 4; ++r) cv[r] = cost[at(wm, r)];
    }
    Place w = wl;
    Two<R> t;
    t.acc = 0.0;
    t.sig2 = 1.0;
    t.f2 = a.fac_b * a.fac_b;
    if constexpr (kOne || MODE == kTurn) {
        One<R> s;
        if (MODE == kFwd && (a.flags & kInit)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s.f[r].x = (R)a.amp0;
                s.f[r].y = (R)0;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) s.f[r] = psi[at(wl, r)];
        }
        if (phaseIn) {
            const auto PK = phase_consts<R>(-a.gamma_in);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                R c, sn;
                phase_cs<true>(-a.gamma_in, cin[r], c, sn, PK);
                s.f[r] = cmul(s.f[r], c, sn);
            }
        }
        s.m = (R)a.mul_f;
        mix_a<M, false, TM>(s, w, mask);
        turn_to<M>(s, w, m, tid);
        mix_b<M, TM>(s, w);
        const R f = (R)a.scl_f;
#pragma unroll
        for (int r = 0; r < 4; ++r) s.f[r] = vscale(s.f[r], f);
        if constexpr (MODE == kFwd) {
            if (wantE) {
#pragma unroll
                for (int r = 0; r < 4; ++r) accE += (double)cv[r] * norm2(s.f[r]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) psi[at(wm, r)] = s.f[r];
        } else if constexpr (MODE == kFwdFuse) {
            const auto PK = phase_consts<R>(-a.gamma_in);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                R c, sn;
                phase_cs<true>(-a.gamma_in, cv[r], c, sn, PK);
                s.f[r] = cmul(s.f[r], c, sn);
            }
            s.m = (R)a.mul_f2;
            mix_b<M, TM2>(s, w);
            turn_to<M>(s, w, m, tid);
            mix_a<M, false, TM2>(s, w, mask);
            const R f2 = (R)a.scl_f2;
#pragma unroll
            for (int r = 0; r < 4; ++r) psi[at(we, r)] = vscale(s.f[r], f2);
        } else {
            // E, lam = C phi; the group is undone on both (phi in memory is the one before it)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                accE += (double)cv[r] * norm2(s.f[r]);
                t.f[r] = s.f[r];
                t.l[r] = vscale(s.f[r], (R)cv[r]);
            }
            t.m = (R)a.mul_b;
            mix_b<M, TM>(t, w);
            turn_to<M>(t, w, m, tid);
            mix_a<M, false, TM>(t, w, mask);
            const R fb = (R)a.scl_b;
#pragma unroll
            for (int r = 0; r < 4; ++r) lam[at(we, r)] = vscale(t.l[r], fb);
        }
    } else {
        const bool from_c = MODE == kBwd && (a.flags & kLamFromC);
#pragma unroll
        for (int r = 0; r < 4; ++r) t.f[r] = psi[at(wl, r)];
        if (from_c) {
#pragma unroll
            for (int r = 0; r < 4; ++r) t.l[r] = vscale(t.f[r], (R)cost[at(wl, r)]);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) t.l[r] = lam[at(wl, r)];
        }
        t.m = (R)a.mul_b;
        mix_a<M, false, TM>(t, w, mask);
        turn_to<M>(t, w, m, tid);
        mix_b<M, TM>(t, w);
        const R f = (R)a.scl_b;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            t.f[r] = vscale(t.f[r], f);
            t.l[r] = vscale(t.l[r], f);
        }
        if (phaseOut) {
            // the last sweep stores nothing, so it skips the phase undo
            const bool undo = kFuse || !(a.flags & kNoStore);
            const auto PK = phase_consts<R>(a.gamma_out);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                accG += (double)cv[r] * imcx(t.l[r], t.f[r]);
                if (undo) {
                    R c, sn;
                    phase_cs<true>(a.gamma_out, cv[r], c, sn, PK);
                    t.f[r] = cmul(t.f[r], c, sn);
                    t.l[r] = cmul(t.l[r], c, sn);
                }
            }
        }
        if constexpr (kFuse) {
            const double acc1 = t.acc;
            t.acc = 0.0;
            t.sig2 = 1.0;
            t.f2 = a.fac_b2 * a.fac_b2;
            t.m = (R)a.mul_b2;
            mix_b<M, TM2>(t, w);
            turn_to<M>(t, w, m, tid);
            mix_a<M, false, TM2>(t, w, mask);
            accB2 = t.acc;
            t.acc = acc1;
            const R f2 = (R)a.scl_b2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                psi[at(we, r)] = vscale(t.f[r], f2);
                lam[at(we, r)] = vscale(t.l[r], f2);
            }
        } else if (!(a.flags & kNoStore)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                psi[at(wm, r)] = t.f[r];
                lam[at(wm, r)] = t.l[r];
            }
        }
    }
    if constexpr (!kOne || MODE == kFwd) {
        if (MODE == kFwd && !wantE) return;
        const double x[4] = {accE, t.acc, accG, accB2};
        const bool want[4] = {wantE, !kOne, phaseOut, MODE == kBwdFuse};
        double sum[4];
        block_sums4<NW>(x, want, m.red, sum);
        if (tid == 0) {
            if (wantE) a.part_e[b] = sum[0];
            if (!kOne) a.part_b[b] = (a.flags & kBetaAcc) ? a.part_b[b] + sum[1] : sum[1];
            if (phaseOut) a.part_g[b] = sum[2];
            if (MODE == kBwdFuse) a.part_b2[b] = (a.flags & kBetaAcc2) ? a.part_b2[b] + sum[3] : sum[3];
        }
    }
}

template <typename R, int M, int MODE, bool TM, bool TM2>
__global__ __launch_bounds__((1 << M) / 4) void k_quad(PassArgs a)
{
    __shared__ QuadLds<R, M> m;
    quad_body<R, M, MODE, TM, TM2>(a, m);
}

template <typename R, int M>
hipError_t launch_quad_m(int mode, const PassArgs &a, unsigned nblocks, hipStream_t s)
{
    const dim3 grid(nblocks), block((1 << M) / 4);
#define QK_ONE(MODE)                                                                              \
    if (a.tan_mode) hipLaunchKernelGGL((k_quad<R, M, MODE, true, true>), grid, block, 0, s, a);   \
    else hipLaunchKernelGGL((k_quad<R, M, MODE, false, false>), grid, block, 0, s, a);            \
    break
#define QK_TWO(MODE)                                                                                              \
    if (a.tan_mode && a.tan_mode2) hipLaunchKernelGGL((k_quad<R, M, MODE, true, true>), grid, block, 0, s, a);    \
    else if (a.tan_mode) hipLaunchKernelGGL((k_quad<R, M, MODE, true, false>), grid, block, 0, s, a);             \
    else if (a.tan_mode2) hipLaunchKernelGGL((k_quad<R, M, MODE, false, true>), grid, block, 0, s, a);            \
    else hipLaunchKernelGGL((k_quad<R, M, MODE, false, false>), grid, block, 0, s, a);                            \
    break
    switch (mode) {
    case kFwd: QK_ONE(kFwd);
    case kTurn: QK_ONE(kTurn);
    case kBwd: QK_ONE(kBwd);
    case kFwdFuse: QK_TWO(kFwdFuse);
    case kBwdFuse: QK_TWO(kBwdFuse);
    default: return hipErrorInvalidValue;
    }
#undef QK_ONE
#undef QK_TWO
    return hipGetLastError();
}

}  // namespace

template <typename R>
hipError_t launch_quad_real(int mode, int tbits, const PassArgs &a, uint64_t nblocks, hipStream_t s)
{
    // what the kernels assume: a full tile whose upper bits are all rotated
    if ((int)a.geo.tbits != tbits || (a.geo.tmask >> 8) != ((1u << tbits) - 1u) >> 8) return hipErrorInvalidValue;
    switch (tbits) {
    case 10: return launch_quad_m<R, 10>(mode, a, (unsigned)nblocks, s);
    case 11: return launch_quad_m<R, 11>(mode, a, (unsigned)nblocks, s);
    case 12: return launch_quad_m<R, 12>(mode, a, (unsigned)nblocks, s);
    default: return hipErrorInvalidValue;
    }
}
#if QK_PASS_MANY
namespace {
// many instances (k_many_pass): every rotation in the tan form
template <int M, int MODE>
__global__ __launch_bounds__((1 << M) / 4) void k_many_quad(PassArgs a, ManyArgs n)
{
    __shared__ QuadLds<double, M> m;
    many_args(a, n);
    quad_body<double, M, MODE, true, true>(a, m);
}
template <int M>
hipError_t launch_many_quad_m(int mode, const PassArgs &a, const ManyArgs &m, dim3 grid, hipStream_t s)
{
    const dim3 block((1 << M) / 4);
    switch (mode) {
    case kFwd: hipLaunchKernelGGL((k_many_quad<M, kFwd>), grid, block, 0, s, a, m); break;
    case kTurn: hipLaunchKernelGGL((k_many_quad<M, kTurn>), grid, block, 0, s, a, m); break;
    case kBwd: hipLaunchKernelGGL((k_many_quad<M, kBwd>), grid, block, 0, s, a, m); break;
    case kFwdFuse: hipLaunchKernelGGL((k_many_quad<M, kFwdFuse>), grid, block, 0, s, a, m); break;
    case kBwdFuse: hipLaunchKernelGGL((k_many_quad<M, kBwdFuse>), grid, block, 0, s, a, m); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_many_quad(int mode, int tbits, const PassArgs &a, const ManyArgs &m, uint64_t nblocks, unsigned count,
                            hipStream_t s)
{
    if ((int)a.geo.tbits != tbits || (a.geo.tmask >> 8) != ((1u << tbits) - 1u) >> 8) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nblocks, count);
    switch (tbits) {
    case 10: return launch_many_quad_m<10>(mode, a, m, grid, s);
    case 11: return launch_many_quad_m<11>(mode, a, m, grid, s);
    case 12: return launch_many_quad_m<12>(mode, a, m, grid, s);
    default: return hipErrorInvalidValue;
    }
}
#endif
template hipError_t launch_quad_real<QK_QUAD_REAL>(int, int, const PassArgs &, uint64_t, hipStream_t);

}  // namespace qk
