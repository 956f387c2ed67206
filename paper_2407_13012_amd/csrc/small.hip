// Expectation and adjoint gradient of a state of at most 4096 stored amplitudes
// (n <= 12, MaxCut n <= 13) in one launch of one workgroup.
//
// Such a gradient used to be 2p + 1 launches of one tile each: 17 + 9 + 8 us of
// kernels at n = 12, p = 2, whose 256 threads left every SIMD one wave to wait
// with, and about 2 us between launches.  Here the state and the adjoint vector
// stay in the registers of up to 1024 threads (4 amplitudes each, 4 waves per
// SIMD) through all layers, MaxCut states folded from n = 9 on, so half of the
// arithmetic goes.  n = 12 (unit MaxCut),
// p = 2, complex128: 14.8 us, the call 60.7 -> 36.7 us.
//
// Layout.  Position p = lane (bits 0-5), register (6-7), wave (8..).  Within a
// wave bits 0-3 are rotated through DPP moves, 6-7 in registers, and 4-5 after
// v_permlane16/32_swap has exchanged them with 6-7 (two instructions per
// amplitude where a lane exchange costs four moves).  The wave bits need LDS:
// in arrangement A element e sits at position e, in B the positions are rotated
// by the number h of wave bits, which puts them at positions 8-h .. 7.  A layer
// starts in the arrangement the last one ended in, so it has one exchange.  The
// partner across bit n-1 of a folded state is the complement ~e; it is read
// during the exchange, from the same LDS image.
//
// Every rotation is in the tan form: exp(-i b X) = -i sin b X (1 + i cot b X)
// where |sin b| > |cos b|, and the flip X of all qubits only exchanges z and ~z
// (nothing at all for a folded state); `flip` tracks it in the cost index.
#include "tile_device.h"

namespace qk {
namespace {

template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Amplitude of lane l ^ (1 << BIT), BIT < 4.
template <int BIT, typename V>
__device__ __forceinline__ V lane_x(V v)
{
    constexpr int kQuad1 = 0xB1, kQuad2 = 0x4E, kQuad3 = 0x1B, kHalfMirror = 0x141, kRor8 = 0x128;
    V o;
    if constexpr (BIT == 0) {
        o.x = dpp<kQuad1>(v.x);
        o.y = dpp<kQuad1>(v.y);
    } else if constexpr (BIT == 1) {
        o.x = dpp<kQuad2>(v.x);
        o.y = dpp<kQuad2>(v.y);
    } else if constexpr (BIT == 2) {  // l ^ 7, then l ^ 3
        o.x = dpp<kQuad3>(dpp<kHalfMirror>(v.x));
        o.y = dpp<kQuad3>(dpp<kHalfMirror>(v.y));
    } else {
        o.x = dpp<kRor8>(v.x);
        o.y = dpp<kRor8>(v.y);
    }
    return o;
}

// Exchanges the bit that tells a from b with lane bit 4 (WIDE: 5).
template <bool WIDE>
__device__ __forceinline__ void swap32(uint32_t &a, uint32_t &b)
{
    if constexpr (WIDE) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
template <bool WIDE>
__device__ __forceinline__ void swap_lane(float &a, float &b)
{
    uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    swap32<WIDE>(x, y);
    a = __builtin_bit_cast(float, x);
    b = __builtin_bit_cast(float, y);
}
template <bool WIDE>
__device__ __forceinline__ void swap_lane(double &a, double &b)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, a), v = __builtin_bit_cast(uint64_t, b);
    uint32_t ul = (uint32_t)u, uh = (uint32_t)(u >> 32), vl = (uint32_t)v, vh = (uint32_t)(v >> 32);
    swap32<WIDE>(ul, vl);
    swap32<WIDE>(uh, vh);
    a = __builtin_bit_cast(double, ((uint64_t)uh << 32) | ul);
    b = __builtin_bit_cast(double, ((uint64_t)vh << 32) | vl);
}
// Positions 6 and 7 <-> 4 and 5.
template <typename V>
__device__ __forceinline__ void swap_quad(V (&v)[4])
{
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        swap_lane<false>(v[k].x, v[k + 1].x);
        swap_lane<false>(v[k].y, v[k + 1].y);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        swap_lane<true>(v[k].x, v[k + 2].x);
        swap_lane<true>(v[k].y, v[k + 2].y);
    }
}

// The rotations of one layer as they are applied: one vector (forward), or both
// with the <lam|X|phi> terms taken before each rotation (adjoint).
template <typename R>
struct One {
    using V = typename Tr<R>::V;
    V f[4];
    R m;
    template <int Q>
    __device__ __forceinline__ void reg()
    {
        bfly<true>(f[0], f[Q ? 2 : 1], m);
        bfly<true>(f[Q ? 1 : 2], f[3], m);
    }
    template <int BIT>
    __device__ __forceinline__ void lane()
    {
#pragma unroll
        for (int r = 0; r < 4; ++r) bfly_lane<true>(f[r], lane_x<BIT>(f[r]), m);
    }
    __device__ __forceinline__ void swap() { swap_quad(f); }
};

template <typename R>
struct Two {
    using V = typename Tr<R>::V;
    V f[4], l[4];
    R m;
    double acc, sig2, f2;
    __device__ __forceinline__ void add(typename PairSum<V>::T ps)
    {
        acc = fma(sig2, (double)ps, acc);
        asm volatile("" : "+v"(acc));
        sig2 *= f2;
    }
    template <int Q>
    __device__ __forceinline__ void reg()
    {
        constexpr int a0 = 0, a1 = Q ? 2 : 1, b0 = Q ? 1 : 2, b1 = 3;
        typename PairSum<V>::T ps = 0;
        ps = imcx_acc(l[a1], f[a0], imcx_acc(l[a0], f[a1], ps));
        ps = imcx_acc(l[b1], f[b0], imcx_acc(l[b0], f[b1], ps));
        add(ps);
        bfly<true>(l[a0], l[a1], m);
        bfly<true>(f[a0], f[a1], m);
        bfly<true>(l[b0], l[b1], m);
        bfly<true>(f[b0], f[b1], m);
    }
    template <int BIT>
    __device__ __forceinline__ void lane()
    {
        typename PairSum<V>::T ps = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const V fp = lane_x<BIT>(f[r]), lp = lane_x<BIT>(l[r]);
            ps = imcx_acc(l[r], fp, ps);
            bfly_lane<true>(l[r], lp, m);
            bfly_lane<true>(f[r], fp, m);
        }
        add(ps);
    }
    __device__ __forceinline__ void swap()
    {
        swap_quad(f);
        swap_quad(l);
    }
};

// Where a thread's amplitudes are: arrangement (0 A, 1 B) and whether positions
// 6-7 and 4-5 are exchanged.  Uniform.
struct Place {
    int arr, sw;
};

// Element of register r.
template <int M>
__device__ __forceinline__ uint32_t elem_at(Place w, uint32_t tid, uint32_t r)
{
    constexpr int H = M > 8 ? M - 8 : 0;
    const uint32_t lane = tid & 63u;
    const uint32_t p = (w.sw ? ((lane & 15u) | (r << 4) | ((lane >> 4) << 6)) : (lane | (r << 6))) | ((tid >> 6) << 8);
    return w.arr ? ((p << H) | (p >> (M - H))) & ((1u << M) - 1u) : p;
}
// LDS slot of an element: strides 1 (A) and 2^H (B) over the lanes hit distinct banks.
template <int M>
__device__ __forceinline__ uint32_t slot_of(uint32_t e)
{
    constexpr int H = M > 8 ? M - 8 : 0;
    return H ? e + (e >> H) : e;
}
template <int M>
constexpr int kSmallSlots = (1 << M) + (M > 8 ? (1 << M) >> (M - 8) : 0);

// Rotates positions [0, bits) of A (bits = 8 except in the M = 8 kernel).
template <int M, typename S>
__device__ __forceinline__ void mix_a(S &s, Place &w, int bits)
{
    // positions 6-7 (sw: 4-5) are in the registers
    const int q0 = w.sw ? 4 : 6;
    if (M > 8 || q0 < bits) s.template reg<0>();
    if (M > 8 || q0 + 1 < bits) s.template reg<1>();
    s.swap();
    w.sw ^= 1;
    const int q1 = w.sw ? 4 : 6;
    if (M > 8 || q1 < bits) s.template reg<0>();
    if (M > 8 || q1 + 1 < bits) s.template reg<1>();
    if (M > 8 || 0 < bits) s.template lane<0>();
    if (M > 8 || 1 < bits) s.template lane<1>();
    if (M > 8 || 2 < bits) s.template lane<2>();
    if (M > 8 || 3 < bits) s.template lane<3>();
}
// Rotates positions 8-H .. 7 of B.
template <int M, typename S>
__device__ __forceinline__ void mix_b(S &s, Place &w)
{
    constexpr int H = M > 8 ? M - 8 : 0;
    if constexpr (H == 1) s.template reg<1>();
    if constexpr (H == 2 || H == 4) {
        s.template reg<0>();
        s.template reg<1>();
    }
    if constexpr (H == 3) {  // 5, 6, 7
        if (!w.sw) s.template reg<0>();
        s.template reg<1>();
    }
    if constexpr (H >= 3) {
        s.swap();
        w.sw ^= 1;
    }
    if constexpr (H == 3) {
        if (!w.sw) s.template reg<0>();
        s.template reg<1>();
    }
    if constexpr (H == 4) {
        s.template reg<0>();
        s.template reg<1>();
    }
}

template <int M, typename V>
__device__ __forceinline__ void put(const V (&v)[4], V *buf, Place w, uint32_t tid)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) buf[slot_of<M>(elem_at<M>(w, tid, r))] = v[r];
}
template <int M, typename V>
__device__ __forceinline__ void get(V (&v)[4], const V *buf, Place w, uint32_t tid, uint32_t flip)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = buf[slot_of<M>(elem_at<M>(w, tid, r) ^ flip)];
}

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
                                          bool folded, int bits)
{
    if (M == 8 || w.arr == 0) {
        mix_a<M>(s, w, bits);
        exchange<M>(s, w, b0, b1, tid, folded);
        if (M > 8) mix_b<M>(s, w);
    } else {
        mix_b<M>(s, w);
        exchange<M>(s, w, b0, b1, tid, folded);
        mix_a<M>(s, w, bits);
    }
}

template <typename R, int M, bool NEAR>
__global__ __launch_bounds__((1 << M) / 4) void k_small_gradient(SmallArgs a, const typename Tr<R>::CT *cost, double *out)
{
    using V = typename Tr<R>::V;
    using CT = typename Tr<R>::CT;
    constexpr int NW = (1 << M) / 256;
    __shared__ V b0[kSmallSlots<M>], b1[kSmallSlots<M>];
    __shared__ double red[2 * kSmallMaxLayers + 1][NW];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const bool folded = a.folded != 0;
    const int bits = M > 8 ? 8 : a.bits, p = a.p;
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
            mix_layer<M, R>(s, w, b0, b1, tid, folded, bits);
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
        mix_layer<M, R>(t, w, b0, b1, tid, folded, bits);
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
