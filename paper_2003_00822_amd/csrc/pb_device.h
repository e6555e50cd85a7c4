// Internal: device functions that the product kernels share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pb {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Cycles that an instruction of the vector ALU takes where two waves or more of a SIMD issue them (profiles/vector_alu_issue.txt): 2.4 to 2.6 for
// V_AND_B32, V_OR_B32, V_XOR_B32, V_MOV_B32, V_ADD_U32 and V_LSHRREV_B32 of vector registers, 2.5 to 4 for V_BITOP3_B32 and V_FMA_F32, by the
// registers that they read; 4.2 to 4.5 with a scalar register, and for V_BFI_B32, V_PERM_B32, V_AND_OR_B32, V_LSHL_OR_B32, V_LSHLREV_B32 and the
// shifts of 64 bits: two registers next to each other are shifted up for the price of one, where what crosses from one to the other is
// masked away.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v)
{
    uint32_t r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));   // (the compiler would use the constant itself)
    return r;
}
template <int N>
__device__ __forceinline__ uint64_t up(uint64_t v)      // v << N (the compiler takes the shifts apart again)
{
    uint64_t r;
    asm("v_lshlrev_b64 %0, %1, %2" : "=v"(r) : "n"(N), "v"(v));
    return r;
}
template <int N>
__device__ __forceinline__ uint64_t down(uint64_t v)    // v >> N
{
    uint64_t r;
    asm("v_lshrrev_b64 %0, %1, %2" : "=v"(r) : "n"(N), "v"(v));
    return r;
}

// x_q = Int(x * 2^f) as a k-bit two's-complement value: toward zero, saturating, NaN -> 0.  V_CVT_I32_F32 does
// exactly that for k = 32 (out-of-range inputs saturate, NaN converts to 0); narrower k clamp the integer.
template <bool NARROW>
__device__ __forceinline__ int32_t to_fixed_point(float x, float fscale, int32_t imin, int32_t imax)
{
    int32_t r;
    const float p = x * fscale;   // exact: a power of two
    asm("v_cvt_i32_f32 %0, %1" : "=v"(r) : "v"(p));
    if constexpr (NARROW)
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(r), "v"(imin), "v"(imax));   // imin <= imax: the clamp
    return r;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}

// LSTM cell update by the four lanes of a quad, which hold the pre-activations y of the gates i, f, g, o of one unit.
// Every lane applies its own gate's nonlinearity (the logistic function as 0.5 tanh(y / 2) + 0.5: one evaluation per
// lane, side by side); the new states are right in the first lane of the quad.
__device__ __forceinline__ void lstm_quad(float y, int lane, float c_old, float *c_new, float *h_new)
{
    const bool is_g = (lane & 3) == 2;
    const float th = tanhf(is_g ? y : 0.5f * y);
    const float act = is_g ? th : fmaf(0.5f, th, 0.5f);
    const float gi = __uint_as_float(dpp_mov<0x00>(__float_as_uint(act)));
    const float gf = __uint_as_float(dpp_mov<0x55>(__float_as_uint(act)));
    const float gg = __uint_as_float(dpp_mov<0xAA>(__float_as_uint(act)));
    const float go = __uint_as_float(dpp_mov<0xFF>(__float_as_uint(act)));
    *c_new = fmaf(gf, c_old, gi * gg);
    *h_new = go * tanhf(*c_new);
}

}  // namespace pb
