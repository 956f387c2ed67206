// Sweeps over many instances at once (batched engine): blockIdx.y is the
// instance, blockIdx.x its tile.
#pragma once
#include "tile_device.h"

namespace qk {
namespace {

__device__ __forceinline__ double uni_d(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// This workgroup's instance filled into the pass arguments.
__device__ __forceinline__ void many_args(PassArgs &a, const ManyArgs &m)
{
    const uint64_t y = blockIdx.y;
    a.psi = (double2 *)a.psi + y * m.stride;
    a.lam = (double2 *)a.lam + y * m.stride;
    a.cost = (const double *)a.cost + y * m.stride;
    a.part_e += y * m.tiles;
    a.part_b += y * m.tiles;
    a.part_g += y * m.tiles;
    a.part_b2 += y * m.tiles;
    const LayerCoef *c = m.coef + y * (uint64_t)m.p;
    const int k = popc(a.geo.tmask);
    const LayerCoef &c1 = c[m.layer];
    a.mul_f = uni_d(c1.mul);
    a.mul_b = -a.mul_f;
    a.fac_f = a.fac_b = uni_d(c1.fac);
    a.scl_f = a.scl_b = uni_d(upow(a.fac_f, k));
    const LayerCoef &c2 = c[m.layer2];
    a.mul_f2 = uni_d(c2.mul);
    a.mul_b2 = -a.mul_f2;
    a.fac_b2 = uni_d(c2.fac);
    a.scl_f2 = a.scl_b2 = uni_d(upow(a.fac_b2, k));
    a.gamma_in = a.gamma_out = uni_d(c[m.layer_phase].gamma);
}

}  // namespace
}  // namespace qk
