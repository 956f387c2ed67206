// Tiles of 2^M amplitudes (M = 8 .. 12) with four amplitudes per thread, for
// states that do not fill the card: the tile code of tile_device.h gives a tile
// of 4096 amplitudes one wave per SIMD, whose chain of rotations and transposes
// nothing overlaps.
//
// Layout.  Position p = lane (bits 0-5), register (6-7), wave (8..).  Within a
// wave bits 0-3 are rotated through DPP moves, 6-7 in registers, and 4-5 after
// v_permlane16/32_swap has exchanged them with 6-7 (two instructions per
// amplitude where a lane exchange costs four moves).  The wave bits need LDS:
// in arrangement A element e sits at position e; in B positions 8-H .. 7 and
// 8 .. 7+H are exchanged (H wave bits).  In both, lanes 0-3 hold the lowest
// four element bits, so LDS accesses are free of bank conflicts and global ones
// are runs of at least 16 amplitudes.
#pragma once
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
    template <int Q, bool TM>
    __device__ __forceinline__ void reg()
    {
        bfly<TM>(f[0], f[Q ? 2 : 1], m);
        bfly<TM>(f[Q ? 1 : 2], f[3], m);
    }
    template <int BIT, bool TM>
    __device__ __forceinline__ void lane()
    {
#pragma unroll
        for (int r = 0; r < 4; ++r) bfly_lane<TM>(f[r], lane_x<BIT>(f[r]), m);
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
    template <int Q, bool TM>
    __device__ __forceinline__ void reg()
    {
        constexpr int a0 = 0, a1 = Q ? 2 : 1, b0 = Q ? 1 : 2, b1 = 3;
        typename PairSum<V>::T ps = 0;
        ps = imcx_acc(l[a1], f[a0], imcx_acc(l[a0], f[a1], ps));
        ps = imcx_acc(l[b1], f[b0], imcx_acc(l[b0], f[b1], ps));
        add(ps);
        bfly<TM>(l[a0], l[a1], m);
        bfly<TM>(f[a0], f[a1], m);
        bfly<TM>(l[b0], l[b1], m);
        bfly<TM>(f[b0], f[b1], m);
    }
    template <int BIT, bool TM>
    __device__ __forceinline__ void lane()
    {
        typename PairSum<V>::T ps = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const V fp = lane_x<BIT>(f[r]), lp = lane_x<BIT>(l[r]);
            ps = imcx_acc(l[r], fp, ps);
            bfly_lane<TM>(l[r], lp, m);
            bfly_lane<TM>(f[r], fp, m);
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
    if (!w.arr) return p;
    constexpr uint32_t low = (1u << (8 - H)) - 1u, mid = (1u << H) - 1u;
    return (p & low) | (((p >> (8 - H)) & mid) << 8) | (((p >> 8) & mid) << (8 - H));
}

// Rotates the element bits 0-7 of `mask` in A.  ALL: all of them, known at
// compile time.
template <int M, bool ALL, bool TM, typename S>
__device__ __forceinline__ void mix_a(S &s, Place &w, uint32_t mask)
{
    // bits 6-7 (sw: 4-5) are in the registers
    const int q0 = w.sw ? 4 : 6;
    if (ALL || ((mask >> q0) & 1u)) s.template reg<0, TM>();
    if (ALL || ((mask >> (q0 + 1)) & 1u)) s.template reg<1, TM>();
    s.swap();
    w.sw ^= 1;
    const int q1 = w.sw ? 4 : 6;
    if (ALL || ((mask >> q1) & 1u)) s.template reg<0, TM>();
    if (ALL || ((mask >> (q1 + 1)) & 1u)) s.template reg<1, TM>();
    if (ALL || (mask & 1u)) s.template lane<0, TM>();
    if (ALL || (mask & 2u)) s.template lane<1, TM>();
    if (ALL || (mask & 4u)) s.template lane<2, TM>();
    if (ALL || (mask & 8u)) s.template lane<3, TM>();
}
// Rotates the element bits 8 .. 7+H (positions 8-H .. 7) in B.
template <int M, bool TM, typename S>
__device__ __forceinline__ void mix_b(S &s, Place &w)
{
    constexpr int H = M > 8 ? M - 8 : 0;
    if constexpr (H == 1) s.template reg<1, TM>();
    if constexpr (H == 2 || H == 4) {
        s.template reg<0, TM>();
        s.template reg<1, TM>();
    }
    if constexpr (H == 3) {  // 5, 6, 7
        if (!w.sw) s.template reg<0, TM>();
        s.template reg<1, TM>();
    }
    if constexpr (H >= 3) {
        s.swap();
        w.sw ^= 1;
    }
    if constexpr (H == 3) {
        if (!w.sw) s.template reg<0, TM>();
        s.template reg<1, TM>();
    }
    if constexpr (H == 4) {
        s.template reg<0, TM>();
        s.template reg<1, TM>();
    }
}

template <int M, typename V>
__device__ __forceinline__ void put(const V (&v)[4], V *buf, Place w, uint32_t tid)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) buf[elem_at<M>(w, tid, r)] = v[r];
}
template <int M, typename V>
__device__ __forceinline__ void get(V (&v)[4], const V *buf, Place w, uint32_t tid, uint32_t flip)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = buf[elem_at<M>(w, tid, r) ^ flip];
}

}  // namespace
}  // namespace qk
