// Preprocessing kernels (Algorithm 1 of the paper): quantize-round the
// fp32 weights to B-bit two's-complement codes (Section 3.3), split the codes
// into B bitlayers, sign layer first (Section 3.2), and pack 32 columns per word
// (Section 3.4); and the way back (pb_unpack).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pb_kernels.h"

namespace pb {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The quantizers reduce over all weights before anything can be packed.  What those passes leave for the next launch
// lives at the start of `packed`, which the packing kernel overwrites last: 32 sums of the clipping search, then per block the
// partial statistics and the partial sum of the +-1 code (256 bytes and 24 per block), then, if there is room, the histogram of
// the clipping search.  A packed matrix has at least 512 bytes, and with B blocks more than B - 1 KB: a bit for each of more
// than 8192 (B - 1) weights.
constexpr int kClipSteps = 32;
constexpr int kClipBins = 4096;
constexpr int kStatsFloats = 8192;      // weights that a block of the reductions takes at a time (32 per thread)
constexpr int kMaxStatsBlocks = 2048;   // eight workgroups per compute unit
struct Partial {
    float absmax, hi, lo, unused;
};
struct Scratch {
    unsigned long long *clip;      // [kClipSteps] sums of the errors
    Partial *stats;                // [blocks]
    unsigned long long *abssum;    // [blocks]
    double *lower, *upper;         // [kClipSteps] bounds of those sums; null: no room (or no need) for the histogram
    unsigned long long *bins;      // [kClipBins] number of weights (upper 28 bits), sum of their distances from the bin's lower edge
    int blocks;
};
static Scratch scratch_of(void *packed, size_t bytes, size_t n, int blocks)
{
    Scratch s;
    s.blocks = blocks;
    s.clip = static_cast<unsigned long long *>(packed);
    s.stats = reinterpret_cast<Partial *>(s.clip + kClipSteps);
    s.abssum = reinterpret_cast<unsigned long long *>(s.stats + blocks);
    s.lower = reinterpret_cast<double *>(s.abssum + blocks);
    s.upper = s.lower + kClipSteps;
    s.bins = reinterpret_cast<unsigned long long *>(s.upper + kClipSteps);
    if ((size_t)(reinterpret_cast<char *>(s.lower) - static_cast<char *>(packed)) > bytes) s.clip = nullptr;   // (never: above)
    // (up to 2^18 weights the exact sums of all thresholds take less time than two more launches, or as little: whole call
    // without / with the histogram at 2^17 weights 19 / 19 us with 2 bits, 21 / 31 with 8, 22 / 31 with 16; at 2^18 22 / 21,
    // 25 / 31 and 29 / 34.  Then few bits gain and many lose, at 420 000 26 / 22, 27 / 33 and 33 / 40; at 2^20 all gain, 33 / 23,
    // 45 / 39 and 62 / 56.  Beyond 2^27 the fields of a workgroup's bins would overflow)
    const size_t end = (size_t)(reinterpret_cast<char *>(s.bins + kClipBins) - static_cast<char *>(packed));
    if (end > bytes || n <= (1u << 18) || n > (1u << 27)) s.lower = s.upper = nullptr;
    return s;
}

// 32 weights per thread, all in flight together; weights past the end read as `pad`.  One way for full and partial blocks:
// loads of 4 bytes each, with their bounds, for the last block took every pass over the weights 2 us more where their number is
// no multiple of 8192 (363 x 361, whole call 9.9 -> 8.2 us with 8 bits, sign quantizer 13.6 -> 11.7; 3001 x 5003 32.2 -> 27.4).
__device__ __forceinline__ void load_weights(const float *__restrict__ W, size_t n, size_t base, float pad, float (&w)[32])
{
    const size_t left = n - base;
    const int valid = left < (size_t)kStatsFloats ? (int)left : kStatsFloats;
    // (loads past the end return 0, dword by dword)
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(W + base), 0, valid * 4, 0x00020000);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (k * 1024 + (int)threadIdx.x * 4) * 4, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * k + e] = __uint_as_float(v[e]);
    }
    if (valid < kStatsFloats) {
#pragma unroll
        for (int k = 0; k < 32; ++k)
            if ((k >> 2) * 1024 + (int)threadIdx.x * 4 + (k & 3) >= valid) w[k] = pad;
    }
}

// `f` on the weights of this block (NaN: as if absent)
template <typename F>
__device__ __forceinline__ void for_each_weight(const float *__restrict__ W, size_t n, F f)
{
    for (size_t base = (size_t)blockIdx.x * kStatsFloats; base < n; base += (size_t)gridDim.x * kStatsFloats) {
        float w[32];
        load_weights(W, n, base, NAN, w);
#pragma unroll
        for (int k = 0; k < 32; ++k) f(w[k]);
    }
}

// a reduction over a workgroup of WAVES waves, result in every thread
template <int WAVES, typename T, typename F>
__device__ __forceinline__ T block_reduce(T v, T *part, F combine)
{
    for (int off = 32; off > 0; off >>= 1) v = combine(v, __shfl_xor(v, off, 64));
    __syncthreads();   // (`part` may still be read from the reduction before)
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    v = part[threadIdx.x & (WAVES - 1)];
    for (int off = WAVES / 2; off > 0; off >>= 1) v = combine(v, __shfl_xor(v, off, 64));
    return v;
}
template <typename T>
__device__ __forceinline__ T sum_of(T a, T b) { return a + b; }

// the same for the three statistics together, once per kernel: one exchange through LDS
template <int WAVES>
__device__ __forceinline__ Partial reduce_stats(float am, float hi, float lo)
{
    __shared__ float4 part[WAVES];
    auto step = [&](int off) {
        am = fmaxf(am, __shfl_xor(am, off, 64));
        hi = fmaxf(hi, __shfl_xor(hi, off, 64));
        lo = fminf(lo, __shfl_xor(lo, off, 64));
    };
    for (int off = 32; off > 0; off >>= 1) step(off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = make_float4(am, hi, lo, 0.0f);
    __syncthreads();
    const float4 p = part[threadIdx.x & (WAVES - 1)];
    am = p.x; hi = p.y; lo = p.z;
    for (int off = WAVES / 2; off > 0; off >>= 1) step(off);
    return Partial{am, hi, lo, 0.0f};
}

// max |W|, max W and min W in one pass (Section 3.3: the step of every quantizer comes from these; fmaxf and fminf
// drop NaN).  Bound: the read of W; 4096 x 4096: 11.5 us = 5.8 TB/s (43.7 us
// with one load in flight per thread).
// The blocks also clear the sums and the histogram of the clipping search, where they are used.
__global__ __launch_bounds__(256) void k_stats(const float *__restrict__ W, size_t n, int clip_search, Scratch s)
{
    if (clip_search) {
        const int i0 = (int)(blockIdx.x * 256 + threadIdx.x), step = (int)(gridDim.x * 256);
        for (int i = i0; i < kClipSteps; i += step) s.clip[i] = 0ull;
        if (s.lower)
            for (int i = i0; i < kClipBins; i += step) s.bins[i] = 0ull;
    }
    float am = 0.0f, hi = -INFINITY, lo = INFINITY;
    for_each_weight(W, n, [&](float w) {
        w = __builtin_canonicalizef(w);   // (a maximum with a signalling NaN is a NaN)
        am = fmaxf(am, fabsf(w));
        hi = fmaxf(hi, w);
        lo = fminf(lo, w);
    });
    const Partial p = reduce_stats<4>(am, hi, lo);
    if (threadIdx.x == 0) s.stats[blockIdx.x] = p;
}

// the statistics of all blocks, in every thread of a workgroup.  All loads of up to 2048 blocks in flight (past the end the last
// block's once more): one memory latency for 2048 blocks, which every kernel that needs the step waits for first (4096 x 4096,
// 8 bits, whole call: 1.6 us less than one load after the other).
template <int WAVES>
__device__ __forceinline__ Partial all_stats(const Scratch &s)
{
    float am = 0.0f, hi = -INFINITY, lo = INFINITY;
    const float4 *stats = reinterpret_cast<const float4 *>(s.stats);   // absmax, hi, lo, unused
    constexpr int K = kMaxStatsBlocks / (WAVES * 64);
    for (int i = threadIdx.x; i < s.blocks; i += K * WAVES * 64) {
        float4 p[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int at = i + k * WAVES * 64;
            p[k] = stats[at < s.blocks ? at : s.blocks - 1];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            am = fmaxf(am, p[k].x);
            hi = fmaxf(hi, p[k].y);
            lo = fminf(lo, p[k].z);
        }
    }
    return reduce_stats<WAVES>(am, hi, lo);
}

__device__ __forceinline__ int quantize_code(float w, float d, int qmin, int qmax)
{
    float r = rintf(w / d);  // IEEE divide, round half to even
    if (r != r) return 0;
    if (r >= (float)qmax) return qmax;
    if (r <= (float)qmin) return qmin;
    return (int)r;
}

// The division of quantize_code by a multiplication where that cannot change the code.  t = w * (1 / d) differs from the
// rounded quotient by less than |t| 2^-22, so rint(t) is the code's rounding unless t is that close to a half-integer
// (for |t| up to qmax + 2; beyond, both clamp).  `off` is the largest distance of the t's from their integers: above
// `limit` the caller divides: in k_pack, whose waves decide over 256 weights, one wave in 60 with 8 bits, one in 5 with 12 and
// nearly all with 16.
struct Quantizer {
    float d, inv, limit;
    int qmin, qmax;
    __device__ __forceinline__ Quantizer(float step, int bits) : d(step)
    {
        qmax = (1 << (bits - 1)) - 1;
        qmin = -(1 << (bits - 1));
        inv = __fdiv_rn(1.0f, d);
        limit = 0.5f - (float)(qmax + 2) * 0x1p-22f;
        // (a step or an inverse outside the normal range: always divide)
        if (!(d >= 0x1p-125f && d <= 0x1p125f)) limit = -1.0f;
    }
    __device__ __forceinline__ float rounded(float w, float &off) const
    {
        const float t = w * inv, r = rintf(t), f = fabsf(t - r);
        off = fmaxf(off, f);   // (an infinite or NaN weight has no distance: code() is right for it)
        return r;
    }
    __device__ __forceinline__ bool must_divide(float off) const { return !(off <= limit); }
    __device__ __forceinline__ int code(float r) const
    {
        const float c = fminf(fmaxf(r, (float)qmin), (float)qmax);
        return r == r ? (int)c : 0;
    }
};

// trunc(|a| * 2^(30 - e)) for |a| < 2^(e + 1): an integer below 2^31, so that the sums below are exact in 64 bits
// and do not depend on the order of the additions
__device__ __forceinline__ unsigned long long fix30(float a, int e)
{
    const float t = truncf(ldexpf(fabsf(a), 30 - e));
    return (t != t) ? 0ull : (unsigned long long)t;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// 1-bit +-1 code (Section 3.3): sum of |W| for the scale d = mean |W|
__global__ __launch_bounds__(256) void k_abs_sum(const float *__restrict__ W, size_t n, Scratch s)
{
    __shared__ unsigned long long part[4];
    float w[32];   // (the first weights are on their way while the statistics come)
    size_t base = (size_t)blockIdx.x * kStatsFloats;
    load_weights(W, n, base, NAN, w);
    const float M = all_stats<4>(s).absmax;
    const int e = M > 0.0f ? ilogbf(M) : 0;
    unsigned long long sum = 0;
    for (;;) {
#pragma unroll
        for (int k = 0; k < 32; ++k) sum += fix30(w[k], e);
        base += (size_t)gridDim.x * kStatsFloats;
        if (base >= n) break;
        load_weights(W, n, base, NAN, w);
    }
    sum = block_reduce<4>(sum, part, sum_of<unsigned long long>);
    if (threadIdx.x == 0) s.abssum[blockIdx.x] = sum;
}

// ---- Clipping search (Section 3.3): the threshold T_k = max|W| k / 32, k = 1 .. 32, with the smallest summed
// |W - d_k q|.  The sums are exact integers (fix30), 32 of them over all weights: 2.3 ms at 3001 x 5003.  Most thresholds
// can be ruled out from a histogram, rigorously: inside a bin where q does not change and W - d_k q keeps its sign, the sum
// of the errors follows from the number of weights and their sum; in any other bin |W - d_k q| changes by no more than W
// does.  That bounds every sum from both sides (k_clip_hist, k_clip_bounds), and only the thresholds whose lower bound
// does not exceed the smallest upper bound are summed exactly (k_clip_err): of N(0, s) weights 3001 x 5003, one or two of
// the 32 with 2 to 5 bits, ten with 8, half of them from 10 bits on, where a bin holds many steps.  Whole call: 2405 -> 54 us
// where one is left, of which the histogram takes 18 (LDS atomics), statistics, step and packing 29; 85 us where two are, 123
// with 8 bits, 350 with 12 and 16.

// the step of threshold k + 1
__device__ __forceinline__ float clip_step(float M, int k, int bits)
{
    const int qmax = (1 << (bits - 1)) - 1;
    return __fdiv_rn(__fmul_rn(M, __fmul_rn((float)(k + 1), 0.03125f)), (float)(qmax > 0 ? qmax : 1));
}
__device__ __forceinline__ bool finite_nonzero(float M) { return M != 0.0f && M < INFINITY; }

// Weights in units of 2^(e - 30) (2^e <= max|W| < 2^(e + 1)) are integers of 32 bits, the upper 12 of which are the bin.
// One LDS atomic per weight: 24 bits of count over 40 bits of summed distances; at the end one global atomic per bin and
// workgroup (28 and 36 bits, the distances in multiples of 2^12).
__global__ __launch_bounds__(1024) void k_clip_hist(const float *__restrict__ W, size_t n, Scratch s)
{
    __shared__ unsigned long long bins[kClipBins];
    const float M = all_stats<16>(s).absmax;
    if (!finite_nonzero(M)) return;
    const int e = ilogbf(M);
    for (int i = threadIdx.x; i < kClipBins; i += 1024) bins[i] = 0ull;
    __syncthreads();
    auto take = [&](float w) {
        const int u = w != w ? 0 : (int)ldexpf(w, 30 - e);
        atomicAdd(&bins[(u >> 20) + kClipBins / 2], (1ull << 40) | (unsigned long long)(u & 0xFFFFF));
    };
    const size_t n4 = n / 4;
    const float4 *W4 = reinterpret_cast<const float4 *>(W);
    for (size_t base = (size_t)blockIdx.x * 4096; base < n4; base += (size_t)gridDim.x * 4096) {
        float4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const size_t i = base + k * 1024 + threadIdx.x;
            v[k] = W4[i < n4 ? i : 0];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (base + k * 1024 + threadIdx.x < n4) { take(v[k].x); take(v[k].y); take(v[k].z); take(v[k].w); }
    }
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) take(W[n4 * 4 + threadIdx.x]);
    __syncthreads();
    for (int i = threadIdx.x; i < kClipBins; i += 1024) {
        const unsigned long long b = bins[i];
        if (b) atomicAdd(&s.bins[i], (b >> 40 << 36) | (b & ((1ull << 40) - 1)) >> 12);
    }
}

// One workgroup per threshold: bounds of its sum, in the units of fix30.  The slack per weight covers the conversion of
// the weight and of its error to integers (1 each), the roundings of d q and W - d q (below 400) and, in bins with a
// change of q, a quotient that rounds the other way (below 1024); per bin, 2^12 for each of at most 256 workgroups whose
// sum of distances was cut to multiples of 2^12.
__global__ __launch_bounds__(1024) void k_clip_bounds(int bits, Scratch s)
{
    __shared__ double part[16];
    const float M = all_stats<16>(s).absmax;
    const int k = blockIdx.x;
    double lo = 0.0, hi = 0.0;
    if (finite_nonzero(M)) {
        const double d = ldexp((double)clip_step(M, k, bits), 30 - ilogbf(M));
        const double qmax = (double)((1 << (bits - 1)) - 1), qmin = -(double)(1 << (bits - 1));
        const double inv = 1.0 / d;   // (an error of 2^-52 in the quotient: far inside the slack)
        auto q_of = [&](double u) { return fmin(fmax(rint(u * inv), qmin), qmax); };
        for (int i = threadIdx.x; i < kClipBins; i += 1024) {
            const unsigned long long bin = s.bins[i];
            if (bin == 0) continue;
            const double n = (double)(bin >> 36), dist = (double)(bin & ((1ull << 36) - 1)) * 4096.0;
            const double u0 = (double)(i - kClipBins / 2) * 0x1p20, u1 = u0 + 0x1p20;
            const double qa = q_of(u0 - 2048.0), qb = q_of(u1 + 2048.0);
            const double ra = u0 - 2048.0 - d * qa, rb = u1 + 2048.0 - d * qb;
            if (qa == qb && (ra >= 0.0) == (rb >= 0.0)) {
                const double sum = fabs(n * (u0 - d * qa) + dist), slack = n * 1024.0 + 0x1p20;
                lo += fmax(sum - slack, 0.0);
                hi += sum + slack;
            } else {
                const double mid = u0 + 0x1p19, g = fabs(mid - d * q_of(mid));
                lo += n * fmax(g - (0x1p19 + 2048.0), 0.0);
                hi += n * (g + (0x1p19 + 2048.0));
            }
        }
    }
    lo = block_reduce<16>(lo, part, sum_of<double>);
    hi = block_reduce<16>(hi, part, sum_of<double>);
    if (threadIdx.x == 0) {
        s.lower[k] = lo * (1.0 - 1e-9);   // (the sums above are rounded)
        s.upper[k] = hi * (1.0 + 1e-9);
    }
}

// the thresholds that may be the best one, as a mask
__device__ __forceinline__ uint32_t clip_candidates(const Scratch &s)
{
    if (!s.lower) return 0xFFFFFFFFu;
    const int k = threadIdx.x & 31;
    const double lo = s.lower[k];
    double best = s.upper[k];
    for (int off = 16; off > 0; off >>= 1) best = fmin(best, __shfl_xor(best, off, 64));
    return (uint32_t)__ballot(lo <= best);
}

// The exact sums of the candidates, unless there is only one.  Bound: the vector ALU, per weight and candidate 11
// operations, and a division more where one of a lane's 32 quotients comes close to a half-integer (Quantizer): hardly ever
// up to 8 bits, in half of the waves with 10 bits, in all of them with 16.  A thread keeps its 32 weights in registers over
// its candidates; the second dimension of the grid shares the candidates out (launch_quantize_pack).
__global__ __launch_bounds__(256) void k_clip_err(const float *__restrict__ W, size_t n, int bits, Scratch s)
{
    __shared__ unsigned long long sums[kClipSteps];
    const uint32_t candidates = clip_candidates(s);
    if (__popc(candidates) == 1) return;
    const float M = all_stats<4>(s).absmax;
    if (!finite_nonzero(M)) return;
    const int e = ilogbf(M);
    if (threadIdx.x < kClipSteps) sums[threadIdx.x] = 0ull;
    __syncthreads();
    for (size_t base = (size_t)blockIdx.x * kStatsFloats; base < n; base += (size_t)gridDim.x * kStatsFloats) {
        float w[32];
        load_weights(W, n, base, 0.0f, w);   // (a weight 0 has the code 0 and no error)
        // weights and steps in units of 2^(e - 30): every rounding as without, but d q cannot overflow next to the largest float
#pragma unroll
        for (int k = 0; k < 32; ++k) w[k] = ldexpf(w[k], 30 - e);
        for (uint32_t left = candidates; left; left &= left - 1) {
            const int c = __builtin_ctz(left);
            if ((unsigned)c % gridDim.y != blockIdx.y) continue;
            const Quantizer Q(ldexpf(clip_step(M, c, bits), 30 - e), bits);
            const float qmax = (float)Q.qmax, qmin = (float)Q.qmin;
            float off = 0.0f;
            unsigned long long sum = 0;
            auto error = [&](float w, float q) {
                // (the product is rounded before the subtraction: __fmul_rn alone leaves that to the compiler)
#pragma clang fp contract(off)
                const float p = Q.d * q;
                return w - p;
            };
#pragma unroll
            for (int k = 0; k < 32; ++k) {
                const float t = w[k] * Q.inv, r = rintf(t);
                off = fmaxf(off, fabsf(t - r));
                const float err = fabsf(error(w[k], fminf(fmaxf(r, qmin), qmax)));
                uint32_t v;   // (toward zero, NaN -> 0)
                asm("v_cvt_u32_f32 %0, %1" : "=v"(v) : "v"(err));
                sum += v;
            }
            if (Q.must_divide(off)) {
                sum = 0;
#pragma unroll
                for (int k = 0; k < 32; ++k) sum += fix30(error(w[k], (float)quantize_code(w[k], Q.d, Q.qmin, Q.qmax)), 30);
            }
            sum = wave_sum_u64(sum);
            if ((threadIdx.x & 63) == 0) atomicAdd(&sums[c], sum);
        }
    }
    __syncthreads();
    if (threadIdx.x < kClipSteps && sums[threadIdx.x]) atomicAdd(&s.clip[threadIdx.x], sums[threadIdx.x]);
}

// the step d of the chosen quantizer, as the layer scales: scales[bits - 1] = d (-d if bits is 1)
__global__ __launch_bounds__(256) void k_step(Scratch s, int bits, int quantizer, size_t n, float *scales)
{
    __shared__ unsigned long long part[4];
    const Partial st = all_stats<4>(s);
    const float M = st.absmax;
    const int qmax = (1 << (bits - 1)) - 1;
    const float qm = (float)(qmax > 0 ? qmax : 1);
    float d;
    if (quantizer == PB_QUANT_RANGE) {
        d = st.hi > st.lo ? __fdiv_rn(__fsub_rn(st.hi, st.lo), (float)(1 << (bits - 1))) : 1.0f;
    } else if (quantizer == PB_QUANT_SIGN) {
        unsigned long long sum = 0;
        for (int i = threadIdx.x; i < s.blocks; i += 256) sum += s.abssum[i];
        sum = block_reduce<4>(sum, part, sum_of<unsigned long long>);
        const int e = M > 0.0f ? ilogbf(M) : 0;
        d = (float)(ldexp((double)sum, e - 30) / (double)n);
    } else if (quantizer == PB_QUANT_CLIP_SEARCH && M != 0.0f) {
        // (the larger threshold on a tie)
        const uint32_t candidates = clip_candidates(s);
        int best = -1;
        unsigned long long best_err = 0;
        for (int k = kClipSteps - 1; k >= 0; --k)
            if ((candidates >> k & 1) && (best < 0 || s.clip[k] < best_err)) { best = k; best_err = s.clip[k]; }
        d = clip_step(M, best, bits);
    } else {
        d = (M == 0.0f) ? 1.0f : __fdiv_rn(M, qm);
    }
    const int i = threadIdx.x;
    if (i < bits) {
        const float v = d * ldexpf(1.0f, bits - 1 - i);
        scales[i] = (i == 0) ? -v : v;
    }
}

typedef int32_t i32x4_dword __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at a 4-byte boundary

// A tile of the packing kernels: 16 packed rows x 16 words (512 columns), 1 KB per bitlayer.  Lane l = 16 kb + j of a
// wave holds the words 4 kb .. 4 kb + 3 of row j (16 contiguous bytes in every layout; in the tiled ones the lanes'
// pieces follow each other).  Word offset of that piece inside a bitlayer:
__device__ __forceinline__ size_t tile_piece(uint32_t layout, int cwp, int rt, int q, int lane)
{
    if (layout == PB_LAYOUT_ROWMAJOR_V1)
        return (size_t)(rt * kTileRows + (lane & 15)) * (size_t)cwp + (size_t)(q * kChunkWords + 4 * (lane >> 4));
    return ((size_t)rt * (size_t)(cwp / kChunkWords) + (size_t)q) * 256 + (size_t)lane * 4;
}

// The 8 x 8 bit transpose in each of the four bytes of x[0 .. 7]: afterwards bit r of byte k of x[b] is what bit b of
// byte k of x[r] was.
template <int S>
__device__ __forceinline__ void transpose_step(uint32_t (&x)[8])
{
    constexpr uint32_t m = S == 4 ? 0x0F0F0F0Fu : S == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = (i & (S - 1)) | ((i & ~(S - 1)) << 1);
        const uint32_t a = x[r], b = x[r + S];
        x[r] = (a & m) | ((b << S) & ~m);
        x[r + S] = ((a >> S) & m) | (b & ~m);
    }
}
__device__ __forceinline__ void transpose_bytes(uint32_t (&x)[8])
{
    transpose_step<4>(x);
    transpose_step<2>(x);
    transpose_step<1>(x);
}

// Quantize, split into bitlayers, pack.  Bound: the read of W.  A workgroup takes one tile of 16 packed rows x 512
// columns: a lane quantizes four columns of a row at a time (16-byte loads, eight in flight) and leaves the codes in LDS
// byte by byte, where column 8 k + r of a word is byte k of dword r; a thread then owns one word position of the tile:
// it reads the 32 codes of its word and transposes them as bits, which delivers the words of eight bitlayers with 1.5
// operations per weight (a ballot per bitlayer and 64 weights, with a select to keep it, took 0.6 operations per weight
// and BITLAYER and stored 8 bytes at a time).  The stores of a bitlayer are contiguous over the threads.
// PL: bytes of a stored code.  4096 x 4096, 8 bits: 14.4 us = 5.8 TB/s (55.6 us with the ballots and a division per weight).
// ROWS: rows per wave; 4 take the whole tile, 1 takes a quarter of it, for matrices of few tiles (launch_quantize_pack).
template <int PL, int ROWS>
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ W, uint32_t layout, int rows, int cols, int bits,
                                              int cwp, int rows_p, int gate_h, size_t layer_words, int quantizer,
                                              const float *__restrict__ scales, uint32_t *__restrict__ packed)
{
    constexpr int kRowBytes = 512 + 16;   // (16 more, so that the rows of a word column start in different banks)
    constexpr int NR = 4 * ROWS;          // rows of the workgroup: NR blockIdx.y .. of the tile
    __shared__ __align__(16) uint8_t codes[PL][NR][kRowBytes];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunks = cwp / kChunkWords;
    const int rt = (int)(blockIdx.x / (unsigned)chunks), ch = (int)(blockIdx.x % (unsigned)chunks);
    const int row0 = rt * kTileRows + NR * (int)blockIdx.y;   // first packed row
    u32x4 w4[ROWS][2];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int pr = row0 + wave * ROWS + k;
        const int r = gate_h ? gates_matrix_row(pr, gate_h) : pr;   // matrix row (-1 or >= rows: padding)
        const bool ok = r >= 0 && r < rows;
        // (loads beyond the end of a row, and of absent rows, return 0)
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(W + (ok ? (size_t)r * (size_t)cols : 0)), 0, ok ? cols * 4 : 0, 0x00020000);
#pragma unroll
        for (int half = 0; half < 2; ++half)
            w4[k][half] = __builtin_amdgcn_raw_buffer_load_b128(rs, (ch * 512 + half * 256 + lane * 4) * 4, 0, 0);
    }
    const Quantizer Q(fabsf(scales[bits - 1]), bits);
    const int stored = is_pairs(layout) ? (bits + 1) & ~1 : bits;   // (an odd number of bitlayers is paired with zeros)
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int j = wave * ROWS + k;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            int u[4];
            if (quantizer == PB_QUANT_SIGN) {
                const int pr = row0 + j;
                const int r = gate_h ? gates_matrix_row(pr, gate_h) : pr;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float w = __uint_as_float(w4[k][half][e]);
                    const bool in = r >= 0 && r < rows && ch * 512 + half * 256 + lane * 4 + e < cols;
                    u[e] = !in ? 0 : (w >= 0.0f || w != w) ? 1 : -1;
                }
            } else {
                float off = 0.0f, r[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] = Q.rounded(__uint_as_float(w4[k][half][e]), off);
#pragma unroll
                for (int e = 0; e < 4; ++e) u[e] = Q.code(r[e]);
                if (Q.must_divide(off)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) u[e] = quantize_code(__uint_as_float(w4[k][half][e]), Q.d, Q.qmin, Q.qmax);
                }
            }
            // columns 4 i .. 4 i + 3 of word w: byte i / 2 of the dwords 4 (i % 2) .. + 3
            const int w = half * 8 + (lane >> 3), i = lane & 7;
            const int at = w * 32 + 16 * (i & 1) + (i >> 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t c = (uint32_t)u[e] << (stored - bits);
                codes[0][j][at + 4 * e] = (uint8_t)c;
                if constexpr (PL == 2) codes[1][j][at + 4 * e] = (uint8_t)(c >> 8);
            }
        }
    }
    __syncthreads();
    // thread -> word position: in the order of the block for the tiled layouts, row by row for the row-major one
    // (with a quarter of a tile a wave has all words, and the waves take a byte each)
    const bool rowmajor = layout == PB_LAYOUT_ROWMAJOR_V1;
    const int t = threadIdx.x & (16 * NR - 1);
    const int j = rowmajor ? t >> 4 : (t >> 2) & (NR - 1);
    const int w = rowmajor ? t & 15 : 4 * (t / (4 * NR)) + (t & 3);
    if (row0 + j >= rows_p || (ROWS == 1 && wave >= PL)) return;
    uint32_t *dst = packed + (rowmajor ? (size_t)(row0 + j) * (size_t)cwp + (size_t)(ch * kChunkWords + w)
                                       : (size_t)blockIdx.x * 256 + 64 * (w >> 2) + 4 * (NR * (int)blockIdx.y + j) + (w & 3));
#pragma unroll
    for (int p0 = ROWS == 1 ? 0 : PL - 1; p0 >= 0; --p0) {
        const int p = ROWS == 1 ? wave : p0;
        uint32_t x[8];
        const u32x4 *src = reinterpret_cast<const u32x4 *>(&codes[p][j][w * 32]);
        const u32x4 a = src[0], b = src[1];
#pragma unroll
        for (int r = 0; r < 4; ++r) { x[r] = a[r]; x[4 + r] = b[r]; }
        transpose_bytes(x);
        if (is_pairs(layout)) {
#pragma unroll
            for (int b2 = 6; b2 >= 0; b2 -= 2) {   // bits 8 p + b2 + 1 (upper bitlayer of the pair) and 8 p + b2
                const int layer = stored - 2 - 8 * p - b2;
                if (layer < 0) continue;
                uint32_t even, odd;
                digits_of_pair(layer == 0 ? ~x[b2 + 1] : x[b2 + 1], x[b2], &even, &odd);   // (the sign bitlayer enters as 1 - w)
                dst[(size_t)layer * layer_words] = even;
                dst[(size_t)(layer + 1) * layer_words] = odd;
            }
        } else {
#pragma unroll
            for (int b1 = 7; b1 >= 0; --b1) {
                const int layer = bits - 1 - 8 * p - b1;
                if (layer >= 0) dst[(size_t)layer * layer_words] = x[b1];
            }
        }
    }
}

// Packed words -> int32 codes.  Bound: the 4-byte stores (a code of B bits takes 4 bytes out and B / 8 in).  A workgroup
// takes one tile: the blocks of all bitlayers go to LDS with one 16-byte load per lane, then a lane puts together four
// adjacent columns of a row (a nibble of one word per bitlayer, spread to the low bits of four bytes by one 24-bit
// multiplication, one accumulating shift per bitlayer) and stores them with 16 bytes, a wave 1 KB of one row.
// 8192 x 8192, 8 bits: 64 us = 5.2 TB/s (594 us with a thread per
// element that fetched one word per bitlayer itself).
// ROWS: rows per wave; 4 take the whole tile, 1 takes a quarter of it, for matrices of few tiles (launch_unpack): the words
// of up to 16 bitlayers then come with one load.
template <int BITS, int ROWS>
__global__ __launch_bounds__(256) void k_unpack(const uint32_t *__restrict__ packed, uint32_t layout, int rows, int cols,
                                                int rows_p, int cwp, int gate_h, size_t layer_words,
                                                int32_t *__restrict__ q)
{
    __shared__ __align__(16) uint32_t words[(BITS + 1) / 2 * 2][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunks = (cols + 511) / 512;
    const int rt = (int)(blockIdx.x / (unsigned)chunks), ch = (int)(blockIdx.x % (unsigned)chunks);
    // this thread's piece of the tile's blocks, and the bitlayers (or pairs of them) first, first + step, ..
    const int part = ROWS == 1 ? 4 * (int)blockIdx.y : 0;   // first row of the tile that the workgroup takes
    const int piece = ROWS == 1 ? 16 * ((threadIdx.x >> 2) & 3) + part + (threadIdx.x & 3) : lane;
    const int first = ROWS == 1 ? threadIdx.x >> 4 : wave, step = ROWS == 1 ? 16 : 4;
    const uint32_t *src = packed + tile_piece(layout, cwp, rt, ch, piece);
    const bool stored_row = layout != PB_LAYOUT_ROWMAJOR_V1 || rt * kTileRows + (piece & 15) < rows_p;
    if (is_pairs(layout)) {
        for (int p = first; p < (BITS + 1) / 2; p += step) {
            const u32x4 even = *reinterpret_cast<const u32x4 *>(src + (size_t)(2 * p) * layer_words);
            const u32x4 odd = *reinterpret_cast<const u32x4 *>(src + (size_t)(2 * p + 1) * layer_words);
            u32x4 upper, lower;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t u, l;
                pair_of_digits(even[t], odd[t], &u, &l);
                upper[t] = p == 0 ? ~u : u;   // (bitlayer 0 is stored complemented)
                lower[t] = l;
            }
            *reinterpret_cast<u32x4 *>(&words[2 * p][piece * 4]) = upper;
            *reinterpret_cast<u32x4 *>(&words[2 * p + 1][piece * 4]) = lower;
        }
    } else {
        for (int i = first; i < BITS; i += step)
            *reinterpret_cast<u32x4 *>(&words[i][piece * 4]) =
                stored_row ? *reinterpret_cast<const u32x4 *>(src + (size_t)i * layer_words) : u32x4{0, 0, 0, 0};
    }
    __syncthreads();
    constexpr int HI = BITS > 8 ? BITS - 8 : 0;   // bitlayers of the upper byte
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        const int j = part + wave * ROWS + k;
        const int pr = rt * kTileRows + j;
        const int r = gate_h ? gates_matrix_row(pr, gate_h) : pr;   // matrix row (-1 or >= rows: padding)
        if (r < 0 || r >= rows) continue;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int c = ch * 512 + half * 256 + lane * 4;
            if (c >= cols) continue;
            const int w = half * 8 + (lane >> 3), shift = 4 * (lane & 7);
            const uint32_t *at = &words[0][((w >> 2) * kTileRows + j) * 4 + (w & 3)];
            uint32_t hi = 0, lo = 0;
#pragma unroll
            for (int i = 0; i < BITS; ++i) {
                const uint32_t spread = (uint32_t)__umul24((at[i * 256] >> shift) & 15u, 0x204081u) & 0x01010101u;
                if (i < HI) hi = (hi << 1) | spread;
                else lo = (lo << 1) | spread;
            }
            i32x4_dword v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (HI > 0)
                    v[e] = (int32_t)(hi << (32 - 8 * e - HI)) >> (32 - HI) << 8 | (int32_t)((lo >> (8 * e)) & 0xFFu);
                else
                    v[e] = (int32_t)(lo << (32 - 8 * e - BITS)) >> (32 - BITS);   // sign-extend the B-bit code
            }
            int32_t *dst = q + (size_t)r * (size_t)cols + c;
            if (c + 3 < cols) {
                *reinterpret_cast<i32x4_dword *>(dst) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < cols) dst[e] = v[e];
            }
        }
    }
}

// Up to this many tiles four workgroups share one: fewer workgroups than compute units leave a tile's four rows per wave
// in sequence.  Graph of packing calls, whole tiles / quarters: 128 x 1000, 8 bits 9.2 / 8.1 us, 16 bits 13.6 / 9.1 (11.9
// with the kernel before the tiles); 1024 x 2048 = 256 tiles, 8 bits 10.2 / 9.5; 1000 x 16384 = 2016 tiles, 8 bits 28.2 / 30.4.
// Unpacking: 363 x 361, 1 bit 3.6 / 2.8 us, 16 bits 5.7 / 3.3 (2.8 and 4.7 with a thread per element); 1024 x 2048, 8 bits
// 5.2 / 4.2; 8192 x 64 = 512 tiles, 1 bit 3.4 / 3.6; 1000 x 16384, 8 bits 14.2 / 15.8.
constexpr unsigned kMaxQuarteredTiles = 256;

int launch_quantize_pack(const float *W, const Layout &L, int quantizer, uint32_t *packed, float *scales,
                         hipStream_t st)
{
    const size_t n = (size_t)L.rows * (size_t)L.cols;
    const size_t want = (n + kStatsFloats - 1) / kStatsFloats;
    const int blocks = (int)(want < (size_t)kMaxStatsBlocks ? want : (size_t)kMaxStatsBlocks);
    const Scratch s = scratch_of(packed, packed_bytes(L), n, blocks);
    if (!s.clip) return (int)hipErrorInvalidValue;
    const bool search = quantizer == PB_QUANT_CLIP_SEARCH;
    hipLaunchKernelGGL(k_stats, dim3(blocks), dim3(256), 0, st, W, n, search ? 1 : 0, s);
    if (quantizer == PB_QUANT_SIGN) hipLaunchKernelGGL(k_abs_sum, dim3(blocks), dim3(256), 0, st, W, n, s);
    if (search) {
        if (s.lower) {
            const size_t hblocks = (n + 16383) / 16384;   // (a workgroup per compute unit: each empties 4096 bins at its end)
            hipLaunchKernelGGL(k_clip_hist, dim3((unsigned)(hblocks < 256 ? hblocks : 256)), dim3(1024), 0, st, W, n, s);
            hipLaunchKernelGGL(k_clip_bounds, dim3(kClipSteps), dim3(1024), 0, st, L.bits, s);
        }
        // A workgroup takes 8192 weights, so that up to 2^21 of them leave compute units without one, or with one that has
        // all thresholds to sum: they are shared out until there are two workgroups per unit.  Whole call, one share / this
        // rule: 2^16 weights 56 / 18 us with 4 bits, 203 / 20 with 12, 138 / 20 with 16; 2^20 weights 31 / 30, 104 / 54 and
        // 98 / 56; from 2^22 on there is one share.
        int shares = 1;
        while (shares < kClipSteps && blocks * shares < 512) shares *= 2;
        hipLaunchKernelGGL(k_clip_err, dim3(blocks, shares), dim3(256), 0, st, W, n, L.bits, s);
    }
    hipLaunchKernelGGL(k_step, dim3(1), dim3(256), 0, st, s, L.bits, quantizer, n, scales);
    const unsigned tiles = (unsigned)((L.rows_p + kTileRows - 1) / kTileRows) * (unsigned)(L.cwp / kChunkWords);
    const bool quarters = tiles <= kMaxQuarteredTiles;
    hipLaunchKernelGGL(quarters ? (L.stored_bits > 8 ? k_pack<2, 1> : k_pack<1, 1>)
                                : (L.stored_bits > 8 ? k_pack<2, 4> : k_pack<1, 4>),
                       dim3(tiles, quarters ? 4 : 1), dim3(256), 0, st, W, L.layout, L.rows, L.cols, L.bits, L.cwp, L.rows_p,
                       L.gate_h, L.layer_words, quantizer, scales, packed);
    return (int)hipGetLastError();
}

int launch_unpack(const uint32_t *packed, const Layout &L, int32_t *q, hipStream_t st)
{
    typedef void (*Unpack)(const uint32_t *, uint32_t, int, int, int, int, int, size_t, int32_t *);
    // (whole tiles, quarters of tiles)
#define PB_UNPACK(B) {k_unpack<B, 4>, k_unpack<B, 1>}
    static const Unpack by_bits[PB_MAX_BITS][2] = {
        PB_UNPACK(1), PB_UNPACK(2), PB_UNPACK(3), PB_UNPACK(4), PB_UNPACK(5), PB_UNPACK(6), PB_UNPACK(7), PB_UNPACK(8),
        PB_UNPACK(9), PB_UNPACK(10), PB_UNPACK(11), PB_UNPACK(12), PB_UNPACK(13), PB_UNPACK(14), PB_UNPACK(15), PB_UNPACK(16)};
#undef PB_UNPACK
    const unsigned tiles = (unsigned)((L.rows_p + kTileRows - 1) / kTileRows) * (unsigned)((L.cols + 511) / 512);
    const bool quarters = tiles <= kMaxQuarteredTiles;
    hipLaunchKernelGGL(by_bits[L.bits - 1][quarters], dim3(tiles, quarters ? 4 : 1), dim3(256), 0, st, packed, L.layout,
                       L.rows, L.cols, L.rows_p, L.cwp, L.gate_h, L.layer_words, q);
    return (int)hipGetLastError();
}

}  // namespace pb
