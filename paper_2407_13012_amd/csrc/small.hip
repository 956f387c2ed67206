// Expectation and adjoint gradient of a state of at most 4096 stored amplitudes
// (n <= 12, MaxCut n <= 13) in one launch of one workgroup.
//
// Such a gradient used to be 2p + 1 launches of one tile each: 17 + 9 + 8 us of
// kernels at n = 12, p = 2, whose 256 threads left every SIMD one wave to wait
// with, and about 2 us between launches.  Here the state and the adjoint vector
// stay in the registers of up to 1024 threads (4 amplitudes each, 4 waves per
// SIMD) through all layers, MaxCut states folded from n = 9 on, so half of the
// arithmetic goes.  n = 12 (unit MaxCut),
// p = 2, complex128: 14.8 us, the call 60.7 -> 29 us (with results in pinned memory).
//
// The layout is that of quad.h: bits 0-7 rotate in arrangement A, the wave bits in
// B.  A layer starts in the arrangement the last one ended in, so it has one
// exchange through LDS.  The partner across bit n-1 of a folded state is the
// complement ~e; it is read during the exchange, from the same LDS image.
//
// Every rotation is in the tan form: exp(-i b X) = -i sin b X (1 + i cot b X)
// where |sin b| > |cos b|, and the flip X of all qubits only exchanges z and ~z
// (nothing at all for a folded state); `flip` tracks it in the cost index.
#include "quad.h"

namespace qk {
namespace {

// The other arrangement, and for a folded state the rotation of bit n-1.
template <int M, typename R>
__device__ __forceinline__ void exchange(One<R> &s, Place &w, typename Tr<R>::V *b0, typename Tr<R>::V *, uint32_t tid,
                                         bool folded)
{
    if (M == 8 && !folded) return;
    lds_barrier();
    put<M>(s.f, b0, w, tid);
    lds_barrier();
    w = Place{w.arr ^ 1, 0};
    get<M>(s.f, b0, w, tid, 0u);
    if (folded) {
        typename Tr<R>::V p[4];
        get<M>(p, b0, w, tid, (1u << M) - 1u);
#pragma unroll
        for (int r = 0; r < 4; ++r) bfly_lane<true>(s.f[r], p[r], s.m);
    }
}
template <int M, typename R>
__device__ __forceinline__ void exchange(Two<R> &s, Place &w, typename Tr<R>::V *b0, typename Tr<R>::V *b1, uint32_t tid,
                                         bool folded)
{
    using V = typename Tr<R>::V;
    if (M == 8 && !folded) return;
    lds_barrier();
    put<M>(s.f, b0, w, tid);
    put<M>(s.l, b1, w, tid);
    lds_barrier();
    w = Place{w.arr ^ 1, 0};
    get<M>(s.f, b0, w, tid, 0u);
    get<M>(s.l, b1, w, tid, 0u);
    if (folded) {
        V fp[4], lp[4];
        get<M>(fp, b0, w, tid, (1u << M) - 1u);
        get<M>(lp, b1, w, tid, (1u << M) - 1u);
        typename PairSum<V>::T ps = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            ps = imcx_acc(s.l[r], fp[r], ps);
            bfly_lane<true>(s.l[r], lp[r], s.m);
            bfly_lane<true>(s.f[r], fp[r], s.m);
        }
        s.add(ps);
    }
}

// All rotations of a layer, starting in the arrangement of `w`.
template <int M, typename R, typename S>
__device__ __forceinline__ void mix_layer(S &s, Place &w, typename Tr<R>::V *b0, typename Tr<R>::V *b1, uint32_t tid,
                                          bool folded, uint32_t mask)
{
    if (M == 8 || w.arr == 0) {
        mix_a<M, (M > 8), true>(s, w, mask);
        exchange<M>(s, w, b0, b1, tid, folded);
        if (M > 8) mix_b<M, true>(s, w);
    } else {
        mix_b<M, true>(s, w);
        exchange<M>(s, w, b0, b1, tid, folded);
        mix_a<M, (M > 8), true>(s, w, mask);
    }
}

template <typename R, int M, bool NEAR>
__global__ __launch_bounds__((1 << M) / 4) void k_small_gradient(SmallArgs a, const typename Tr<R>::CT *cost, double *out)
{
    using V = typename Tr<R>::V;
    using CT = typename Tr<R>::CT;
    constexpr int NW = (1 << M) / 256;
    __shared__ V b0[1 << M], b1[1 << M];
    __shared__ double red[2 * kSmallMaxLayers + 1][NW];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const bool folded = a.folded != 0;
    const int p = a.p;
    const uint32_t size = 1u << (M > 8 ? M : a.bits), all = size - 1u;
    Place w{0, 0};
    uint32_t flip = 0;  // all: amplitude e holds index ~e
    CT cv[4];
    auto load_cost = [&] {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t e = elem_at<M>(w, tid, r);
            cv[r] = M > 8 || e < size ? cost[(e ^ flip) & all] : (CT)0;
        }
    };
    Two<R> t;
    {
        One<R> s;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s.f[r].x = M > 8 || elem_at<M>(w, tid, r) < size ? (R)a.amp0 : (R)0;
            s.f[r].y = (R)0;
        }
#pragma nounroll
        for (int l = 0; l < p; ++l) {
            load_cost();
            const auto PK = phase_consts<R>(-a.layer[l].gamma);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                R c, sn;
                phase_cs<NEAR>(-a.layer[l].gamma, cv[r], c, sn, PK);
                s.f[r] = cmul(s.f[r], c, sn);
            }
            s.m = (R)a.layer[l].mul;
            mix_layer<M, R>(s, w, b0, b1, tid, folded, all);
            const R f = (R)a.layer[l].scl;
#pragma unroll
            for (int r = 0; r < 4; ++r) s.f[r] = vscale(s.f[r], f);
            if (a.layer[l].flip && !folded) flip ^= all;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) t.f[r] = s.f[r];
    }
    // E, lam = C phi
    load_cost();
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        acc += (double)cv[r] * norm2(t.f[r]);
        t.l[r] = vscale(t.f[r], (R)cv[r]);
    }
    acc = wave_sum(acc);
    if (lane == 0) red[0][wave] = acc;
#pragma nounroll
    for (int l = p - 1; l >= 0; --l) {
        t.acc = 0.0;
        t.sig2 = 1.0;
        t.f2 = a.layer[l].fac * a.layer[l].fac;
        t.m = (R)-a.layer[l].mul;
        mix_layer<M, R>(t, w, b0, b1, tid, folded, all);
        if (a.layer[l].flip && !folded) flip ^= all;
        load_cost();
        const R f = (R)a.layer[l].scl;
        double g = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            t.f[r] = vscale(t.f[r], f);
            t.l[r] = vscale(t.l[r], f);
            g += (double)cv[r] * imcx(t.l[r], t.f[r]);
        }
        if (l > 0) {
            const auto PK = phase_consts<R>(a.layer[l].gamma);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                R c, sn;
                phase_cs<NEAR>(a.layer[l].gamma, cv[r], c, sn, PK);
                t.f[r] = cmul(t.f[r], c, sn);
                t.l[r] = cmul(t.l[r], c, sn);
            }
        }
        const double bs = wave_sum(t.acc), gs = wave_sum(g);
        if (lane == 0) {
            red[1 + l][wave] = bs;
            red[1 + p + l][wave] = gs;
        }
    }
    __syncthreads();
    for (uint32_t k = tid; k <= 2u * p; k += (1 << M) / 4) {
        double s = red[k][0];
#pragma unroll
        for (int i = 1; i < NW; ++i) s += red[k][i];
        out[k] = folded ? 2.0 * s : s;
    }
}

template <typename R, bool NEAR>
hipError_t launch_m(const SmallArgs &a, const void *cost, double *out, hipStream_t s)
{
    using CT = typename Tr<R>::CT;
    switch (a.bits) {
    case 12: hipLaunchKernelGGL((k_small_gradient<R, 12, NEAR>), dim3(1), dim3(1024), 0, s, a, (const CT *)cost, out); break;
    case 11: hipLaunchKernelGGL((k_small_gradient<R, 11, NEAR>), dim3(1), dim3(512), 0, s, a, (const CT *)cost, out); break;
    case 10: hipLaunchKernelGGL((k_small_gradient<R, 10, NEAR>), dim3(1), dim3(256), 0, s, a, (const CT *)cost, out); break;
    case 9: hipLaunchKernelGGL((k_small_gradient<R, 9, NEAR>), dim3(1), dim3(128), 0, s, a, (const CT *)cost, out); break;
    default:
        if (a.bits < 1 || a.bits > 8) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_small_gradient<R, 8, NEAR>), dim3(1), dim3(64), 0, s, a, (const CT *)cost, out);
    }
    return hipGetLastError();
}

}  // namespace

bool small_fits(int n, bool maxcut, int p)
{
    return n - (small_folds(n, maxcut) ? 1 : 0) <= kSmallBits && p >= 1 && p <= kSmallMaxLayers;
}

SmallArgs small_args(int n, bool maxcut, int p, const double *gamma, const double *beta)
{
    SmallArgs a{};
    a.folded = small_folds(n, maxcut);
    a.bits = n - a.folded;
    a.p = p;
    a.amp0 = 1.0 / sqrt((double)(1ull << n));
    for (int l = 0; l < p; ++l) {
        const double c = cos(beta[l]), s = sin(beta[l]);
        SmallLayer &y = a.layer[l];
        y.gamma = gamma[l];
        y.flip = fabs(c) < fabs(s);
        y.mul = y.flip ? -c / s : s / c;
        y.fac = y.flip ? s : c;
        y.scl = 1.0;
        for (int i = 0; i < n; ++i) y.scl *= y.fac;
    }
    return a;
}

hipError_t launch_small_gradient(bool c64, bool near, const SmallArgs &a, const void *cost, double *out, hipStream_t s)
{
    if (c64) return near ? launch_m<float, true>(a, cost, out, s) : launch_m<float, false>(a, cost, out, s);
    return near ? launch_m<double, true>(a, cost, out, s) : launch_m<double, false>(a, cost, out, s);
}

}  // namespace qk
