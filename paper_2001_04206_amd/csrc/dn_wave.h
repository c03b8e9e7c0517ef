// Wave-level reductions shared by the kernels of this library (64-lane wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

namespace dn {

// Wave-wide reductions with data-parallel-primitive moves (no LDS traffic): butterflies inside
// each row of 16 lanes, then the row totals are carried across rows; lane 63 ends up with the
// result, which is broadcast through a scalar register.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_move(float v, float identity)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, identity),
                                                                 __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf,
                                                                 false));
}

__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_move<0xB1, 0xf>(v, 0.f);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4E, 0xf>(v, 0.f);    // quad_perm [2,3,0,1]
    v += dpp_move<0x141, 0xf>(v, 0.f);   // row_half_mirror
    v += dpp_move<0x140, 0xf>(v, 0.f);   // row_mirror: every lane of a row holds the row's sum
    v += dpp_move<0x142, 0xa>(v, 0.f);   // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v, 0.f);   // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

__device__ __forceinline__ float wave_max(float v)
{
    const float ninf = -INFINITY;
    v = fmaxf(v, dpp_move<0xB1, 0xf>(v, ninf));
    v = fmaxf(v, dpp_move<0x4E, 0xf>(v, ninf));
    v = fmaxf(v, dpp_move<0x141, 0xf>(v, ninf));
    v = fmaxf(v, dpp_move<0x140, 0xf>(v, ninf));
    v = fmaxf(v, dpp_move<0x142, 0xa>(v, ninf));
    v = fmaxf(v, dpp_move<0x143, 0xc>(v, ninf));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Completes this wave's device-scope stores before it signals another workgroup.
// Data that crosses workgroups is written with relaxed device-scope atomic stores, which the
// hardware performs as write-through stores to the level all workgroups of the device share.  A
// wave's memory counter reaches zero only when every store it has issued has been acknowledged
// from that level (the compiler's own code for a device-scope release leans on the same fact), so
// after this call -- and a workgroup barrier, when another wave does the signalling -- a flag or
// counter written with a device-scope atomic is observed only after the data.  The workgroup-scope
// release fence keeps the compiler from sinking stores below the wait.  Unlike a device-scope
// release fence this does not write back the L2, which such stores never leave dirty.
__device__ __forceinline__ void drain_device_scope_stores()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);   // vmcnt, expcnt, lgkmcnt = 0
}

// Sum over each aligned group of 16 lanes (a DPP row); every lane of the group gets it.
__device__ __forceinline__ float row16_sum(float v)
{
    v += dpp_move<0xB1, 0xf>(v, 0.f);
    v += dpp_move<0x4E, 0xf>(v, 0.f);
    v += dpp_move<0x141, 0xf>(v, 0.f);
    v += dpp_move<0x140, 0xf>(v, 0.f);
    return v;
}

// e^x for x <= 0 (NaN stays): 2^n 2^r with x log2 e = n + r, |r| <= 1/2; log2 e in two parts.  n is that of x bounded (NaN: to -150),
// so that it has an integer; the rest of an x below the bound is a power of two that is 0 in fp32.
__device__ __forceinline__ float exp_below_zero(float x)
{
    const float n = __builtin_rintf(__builtin_amdgcn_fmed3f(x, -150.f, 0.f) * 1.44269502f);
    float r = __builtin_fmaf(x, 1.44269502f, -n);
    r = __builtin_fmaf(x, 1.92596299e-8f, r);
    return __builtin_ldexpf(__builtin_amdgcn_exp2f(r), (int)n);
}

// 1 / x of a normal number: the hardware's estimate and one Newton step.
__device__ __forceinline__ float inverse(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.f), r, r);
}

// 1 / (1 + e^-z) (NaN stays): the same two, n of z bounded where the result is 0 or 1 in fp32 anyway.
__device__ __forceinline__ float sigmoid_of(float z)
{
    const float n = __builtin_rintf(__builtin_amdgcn_fmed3f(z, -150.f, 150.f) * -1.44269502f);
    float r = __builtin_fmaf(z, -1.44269502f, -n);
    r = __builtin_fmaf(z, -1.92596299e-8f, r);
    const float d = 1.f + __builtin_ldexpf(__builtin_amdgcn_exp2f(r), (int)n), inv = __builtin_amdgcn_rcpf(d);
    return d < 0x1p100f ? __builtin_fmaf(__builtin_fmaf(-d, inv, 1.f), inv, inv) : inv;
}

}  // namespace dn
