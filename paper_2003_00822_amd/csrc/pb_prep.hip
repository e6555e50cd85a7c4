// Run-time activation processing (Algorithm 2 of the paper, x_q = Int(x * 2^f);
// Section 3.3: "a multiplication and a cast"; Section 3.4: the bitwise matrix
// transpose that lays the bits of one plane next to each other for AND/popcount).
//
// A workgroup of 4 waves owns 256 consecutive columns of one activation vector, a
// lane one column.  The transpose is the wave64 ballot: bit j of the 64 lanes'
// fixed-point values IS two packed words of plane j; lane j keeps ballot j and
// stores it.  32 columns groups of a vector run in parallel on
// different CUs, so the step is launch-latency bound, not compute bound.
// The first workgroup of a vector also finds the plane statistics that let the product kernel skip planes carrying
// no information: h = number of magnitude bits in use (planes h..31 all equal the sign plane and together weigh
// -2^h) and whether any value is negative.  The conversion is monotone, so both follow from the largest and the
// smallest activation: one maximum and one minimum per value instead of a conversion, and the whole vector (8192
// columns at a time) is one round of 16-byte loads, in flight together with the workgroup's own columns.  No
// cross-workgroup reduction or second launch; skipping those planes changes no result bit.
// Bound: launch and one memory latency.  One vector, activations prepared and two products (4 of 8 bitlayers): 4096
// columns, 4096 + 1000 rows 16.9 -> 15.9 us, 8192 columns, 8192 + 4096 rows 33.4 -> 31.2 us (before: every workgroup
// converted the whole vector, 2048 columns of 4-byte loads at a time).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pb_kernels.h"

namespace pb {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// k-bit saturating, toward-zero conversion of p = x * 2^f; NaN -> 0.  lim = 2^(k-1), lim_below = the largest
// float below it.  Branch-free: clamp into the range where the cast is defined, then patch the top end and NaN
// (the bottom end, -2^(k-1), converts exactly).
__device__ __forceinline__ int32_t to_fixed(float p, float lim, float lim_below, int32_t imax)
{
    const float pc = fminf(fmaxf(p, -lim), lim_below);
    int32_t r = (int32_t)pc;
    r = (p >= lim) ? imax : r;
    return (p != p) ? 0 : r;
}

__global__ __launch_bounds__(256) void k_prep(const float *__restrict__ X0, int cols0, const float *__restrict__ X1,
                                              int cols1, int cwp, float fscale, float lim, float lim_below,
                                              int32_t imax, uint32_t *__restrict__ planes, int *__restrict__ meta,
                                              int32_t *__restrict__ xq_out)
{
    __shared__ float s_max[4], s_min[4];
    const int n = blockIdx.y;
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int C = cols0 + cols1;
    const float *x0 = X0 + (size_t)n * cols0;
    const float *x1 = X1 ? X1 + (size_t)n * cols1 : nullptr;

    // this lane's own column first, then, in the first workgroup, the whole vector
    const int c_own = (b << 8) + tid;
    float v_own = 0.0f;
    if (c_own < cols0) v_own = x0[c_own];
    else if (c_own < C) v_own = x1[c_own - cols0];
    float pmax = 0.0f, pmin = 0.0f;   // (fmaxf and fminf drop NaN, which converts to 0)
    auto take = [&](const float *x, int cols) {
        // (loads past the end return 0, dword by dword; rows of any width start at a 4-byte boundary)
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(x), 0, cols * 4, 0x00020000);
        for (int c0 = 0; c0 < cols; c0 += 8192) {
            u32x4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, (c0 + j * 1024 + tid * 4) * 4, 0, 0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __uint_as_float(v[j][e]) * fscale;   // (makes a signalling NaN quiet)
                    pmax = fmaxf(pmax, p);
                    pmin = fminf(pmin, p);
                }
            }
        }
    };
    if (b == 0) {
        take(x0, cols0);
        if (cols1 > 0) take(x1, cols1);
    }
    const int32_t mine = to_fixed(v_own * fscale, lim, lim_below, imax);
    if (xq_out && c_own < C) xq_out[(size_t)n * C + c_own] = mine;

    // bitwise transpose of this wave's 64 columns: ballot j = words (2g, 2g+1) of plane j
    // (a select per plane rather than v_writelane: the compiler then inserts the wait states that a VALU-written
    // SGPR needs before a lane-indexed write reads it)
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const unsigned long long bal = __ballot((mine >> j) & 1);
        lo = (lane == j) ? (uint32_t)bal : lo;
        hi = (lane == j) ? (uint32_t)(bal >> 32) : hi;
    }
    const int word0 = 2 * (4 * b + wave);
    if (lane < 32 && word0 < cwp) {
        uint32_t *dst = planes + ((size_t)n * 32 + lane) * (size_t)cwp + word0;
        *reinterpret_cast<uint2 *>(dst) = make_uint2(lo, hi);
    }

    if (b != 0) return;
    for (int off = 32; off > 0; off >>= 1) {
        pmax = fmaxf(pmax, __shfl_xor(pmax, off, 64));
        pmin = fminf(pmin, __shfl_xor(pmin, off, 64));
    }
    if (lane == 0) { s_max[wave] = pmax; s_min[wave] = pmin; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) {
            pmax = fmaxf(pmax, s_max[w]);
            pmin = fminf(pmin, s_min[w]);
        }
        // the largest magnitude among the non-negative values (v) and among the negative ones (~v)
        const int32_t vmax = to_fixed(pmax, lim, lim_below, imax);
        const int32_t vmin = to_fixed(pmin, lim, lim_below, imax);
        const uint32_t mg = (uint32_t)vmax | (uint32_t)(vmin ^ (vmin >> 31));
        const int h = mg ? 32 - __clz((int)mg) : 0;   // magnitude planes 0..h-1; plane h is the sign plane
        const int neg = vmin < 0;
        const int nplanes = neg ? h + 1 : h;          // planes that must be multiplied
        int *mt = meta + (size_t)n * kMetaInts;
        mt[0] = h;
        mt[1] = neg;
        mt[2] = (nplanes + 3) >> 2;                   // passes of 4 planes
        mt[3] = nplanes;
    }
}

int launch_prep(const float *X0, int cols0, const float *X1, int cols1, int batch, const Layout &L, int frac_bits,
                int act_bits, uint32_t *planes, int *meta, int32_t *xq_out, hipStream_t st)
{
    float fscale = ldexpf(1.0f, frac_bits);
    float lim = ldexpf(1.0f, act_bits - 1);
    int32_t imax = (act_bits == 32) ? INT32_MAX : (int32_t)((1u << (act_bits - 1)) - 1u);
    float lim_below = nextafterf(lim, 0.0f);
    hipLaunchKernelGGL(k_prep, dim3(L.cwp / 8, batch), dim3(256), 0, st, X0, cols0, X1, cols1, L.cwp, fscale, lim,
                       lim_below, imax, planes, meta, xq_out);
    return (int)hipGetLastError();
}

}  // namespace pb
