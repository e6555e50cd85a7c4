// The kernel for one activation vector on the matrix cores: the whole inference path of Algorithm 2 of the
// paper in one launch -- x_q = Int(x * 2^f), the bitwise transpose into bit planes
// (Section 3.4), the 1-bit products of Section 3.1 with the planes of the
// vector batched as the second matrix operand ("one batched matrix product"), the plane
// weights [-2^31, 2^30 .. 2^0] and the scale-accumulation over the first `bits_used`
// bitlayers (the run-time knob of the abstract).  (Batches: pb_imma.hip.)
//
// Why the matrix cores: AND + popcount costs two vector-ALU lane operations per
// (32-bit weight word, plane); with 32 planes that is four times what the ALUs of
// this chip can do while HBM delivers the words.  The same inner products are a
// dense contraction, and V_MFMA_SCALE_F32_16X16X128_F8F6F4 on FP4 (E2M1) operands
// does 32768 multiply-adds per instruction with exact results.
//
// Two planes per operand row.  E2M1 holds 0, 0.5, 1.0 and 1.5 as the codes 0, 1, 2, 3,
// so the two adjacent planes 2 i and 2 i + 1 of the activations travel as ONE row of
// base-4 digits d = b_(2i) + 2 b_(2i+1) (FP4 code = d, value d / 2): the 32 planes of a
// vector are the 16 rows of one A operand and the plane weights become 4^i.  The weight
// bit is the code 2.0, so every product is the digit itself (0 .. 3), the fp32
// accumulators hold integers below 2^24 and every sum is exact.
// The sign plane: digit 15 (bits 31, 30) is the signed one, -2 b_31 + b_30, and E2M1 has
// the values 0, 0.5, -1.0, -0.5 too (codes 0000, 0001, 1010, 1001): the two's-complement
// value is sum_i 4^i digit_i with that one digit signed, nothing to correct afterwards.
//
// Operands.  A (16 x 128) = 16 digit rows x 128 columns, B (128 x 16) = 128 columns x
// 16 weight rows, D (16 x 16): lane l of D holds row j = l % 16 of the weights and
// the operand rows 4 * (l / 16) + c in its four registers c (rows 0-7 carry the even
// digits, rows 8-15 the odd ones, see digit_of_row), so the digit weighting is
// arithmetic inside a lane.  A lane's B operand is 32 columns of one weight row = ONE
// packed word; register r, nibble n of both operands is column 4 n + r of the word:
//     b0 = (w << 2) & 0x44444444   b1 = (w << 1) & 0x44444444
//     b2 = w & 0x44444444          b3 = (w >> 1) & 0x44444444
//
// Mapping.  A wave owns a slice of the columns (NQ chunks of 512) for its whole life
// and keeps the digit rows of that slice in registers; it streams the 1 KB
// blocks of its slice (see pb_layout.h) for row tile after row tile and bitlayer
// after bitlayer with 16-byte loads, several blocks in flight.  The waves of a
// workgroup are the slices of one row; their per-(row, bitlayer) sums meet in LDS
// through integer atomics, once per row tile, and one wave applies the layer scales
// and stores.  All integer results are exact, so they do not depend on the schedule.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <type_traits>

#include "pb_device.h"
#include "pb_kernels.h"

namespace pb {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// The arguments that the first memory requests of a wave depend on are the kernel's leading scalar parameters: those
// (thirteen dwords) the hardware loads into registers before a wave starts (kernel-argument preload), so the requests
// need not wait for a round trip to the argument buffer.  The rest travels as one structure.
struct MfmaHead {
    const uint32_t *packed;
    const float *X0;            // activations: row n is [X0[n][0..cols0) ; X1[n][0..cols1)]
    uint32_t packed_bytes;      // (below 2^32: the blocks are addressed with 32-bit offsets)
    uint32_t flags;             // kPlanesGiven: bit planes already in memory (prepared mode); kSecondPart: X1 is given
    int cols0;
    uint32_t layer_step, round_step;   // bytes from one bitlayer of a row tile to the next, from one row tile to the next
    int rounds_per_wg;          // row tiles per workgroup
    int rt_count, cq;
    int m;                      // bitlayers to accumulate
};
constexpr uint32_t kPlanesGiven = 1, kSecondPart = 2;
struct MfmaArgs {
    const float *X1;
    const uint32_t *planes;     // non-null: bit planes already in memory [32][cwp] (prepared mode)
    const float *scales;
    float *Y;
    long long *A;
    const float *bias;          // [rows] or null: added to the fp32 result
    const float *c_prev;        // non-null: LSTM cell update instead of the store of Y (gate-interleaved rows)
    float *h_out, *c_out;
    int relu;                   // max(., 0) before the store of Y
    int gate_h;                 // gate-interleaved rows: H (packed row 16 t + 4 (u % 4) + gate = row gate * H + u), else 0
    int cols1;
    int R, cwp;
    float fscale;               // 2^frac_bits
    int imin, imax;             // range of the act_bits-bit fixed-point values
    double out_scale;           // 2^-frac_bits
};

// z + (z of the lane D lanes away, D = 16 or 32), in both lanes
template <int D>
__device__ __forceinline__ double add_across(double z)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(z);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    // the swap leaves (own, partner's) in one half of the lanes and (partner's, own) in the other
    const auto l = D == 16 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                           : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = D == 16 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                           : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
           __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// Row order of the A operand.  The sixteen base-4 digits of a value travel as FP4 codes in two words: E = the even
// digits (x & 0x33333333: nibble k = digit 2 k) and O = the odd ones ((x >> 2) & 0x33333333: nibble k = digit
// 2 k + 1).  Operand row i is nibble i of the pair (E, O): rows 0-7 hold the digits 0, 2, .., 14 and rows 8-15 the
// digits 1, 3, .., 15.
__device__ __forceinline__ int digit_of_row(int i) { return ((i & 7) << 1) | (i >> 3); }

// x_q (k-bit two's complement, sign-extended) -> the FP4 codes of its sixteen digits, nibble i = digit
// digit_of_row(i); code = digit (value digit / 2), except for digit 15, the signed one (-2 b31 + b30: values
// 0, 1, -2, -1 = codes 0000, 0001, 1010, 1001), which a byte table indexed by the two top bits supplies.
__device__ __forceinline__ uint2 digit_codes(uint32_t x)
{
    const uint32_t e = x & 0x33333333u;
    const uint32_t o = (x >> 2) & 0x33333333u;
    // the top two bits, as the low bits of a selector byte: byte 3 of x >> 6 is x >> 30.  The selected table
    // byte holds the code in its upper nibble.
    const uint32_t top = __builtin_amdgcn_perm(0u, 0x90A01000u, x >> 6);
    return make_uint2(e, (o & 0x0FFFFFFFu) | (top & 0xF0000000u));
}

// The 16 x 16 transpose of 4-bit elements that the LDS performs on a read (DS_READ_B64_TR_B4): in every group of
// 16 lanes, lane i receives nibble i of the 64-bit rows that the lanes e = 0 .. 15 of its group address, the one
// of lane e in nibble e.
typedef int v2i __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 lds_read_transposed(const uint2 *row)
{
    const v2i r = __builtin_amdgcn_ds_read_tr4_b64_v2i32((v2i __attribute__((address_space(3))) *)(row));
    return make_uint2((uint32_t)r.x, (uint32_t)r.y);
}

// Staging area of one wave for one chunk of 512 columns: 16 words x 32 columns x 8 bytes (the codes of a column).
// The row of column 4 n + r of word w sits at w * 40 + 8 r + n (in units of 8 bytes): the columns of one operand
// register are contiguous; a word takes 320 bytes, so that the 64-byte pieces that the lanes of a write put into
// adjacent words fall into different banks, and every position of a lane is a constant away from its first.
constexpr int kStageRows = 16 * 40;
__device__ __forceinline__ int stage_row(int w, int r, int n) { return w * 40 + 8 * r + n; }

// The same operand from the two plane words (bit c = column c) of a digit row: p0 the lower plane, p1 the upper
__device__ __forceinline__ void digit_operand_from_planes(uint32_t p0, uint32_t p1, u32x4 &dst)
{
    // digits of the even columns c at bits c, c + 1; of the odd columns c at bits c - 1, c
    uint32_t e = (p0 & 0x55555555u) | ((p1 << 1) & ~0x55555555u);
    uint32_t o = ((p0 >> 1) & 0x55555555u) | (p1 & ~0x55555555u);
    asm("" : "+v"(e), "+v"(o));   // (keeps the two words whole: ten operations instead of fourteen)
    dst.x = e & 0x33333333u;
    dst.y = o & 0x33333333u;
    dst.z = (e >> 2) & 0x33333333u;
    dst.w = (o >> 2) & 0x33333333u;
}

// digits (b1 b0) of the top row -> the codes of their signed value -2 b1 + b0; `top` = 0x22222222 in the lanes
// of digit 15, else 0 (then nothing changes)
__device__ __forceinline__ uint32_t signed_top_digit(uint32_t d, uint32_t top)
{
    return (d & ~((d << 1) & top)) | ((d & top) << 2);
}

__device__ __forceinline__ v8i as_operand(const u32x4 v)
{
    v8i r = {(int)v.x, (int)v.y, (int)v.z, (int)v.w, 0, 0, 0, 0};   // FP4 operands use the first four registers
    return r;
}

// Two packed words -> their B operands: FP4 code 2.0 where the weight bit is set.  Register r of an operand holds the columns 4 n + r.
// The shifts are those of both words at once: eleven operations of the vector ALU instead of fourteen (4096 x 4096, 8 bitlayers 4.8 -> 4.6
// us, an LSTM step of 6000 x 3000 with 8 bitlayers 6.8 -> 6.35, 500 x 12001, 16 bitlayers 11.9 -> 11.05).  The constant in a vector register
// measured 0.02 to 0.5 us slower here.
__device__ __forceinline__ void weight_operands(uint64_t w, v8i &b0, v8i &b1)
{
    constexpr uint32_t code = 0x44444444u;
    const uint64_t r0 = up<2>(w), r1 = up<1>(w), r3 = down<1>(w);
    b0 = v8i{(int)((uint32_t)r0 & code), (int)((uint32_t)r1 & code), (int)((uint32_t)w & code), (int)((uint32_t)r3 & code), 0, 0, 0, 0};
    b1 = v8i{(int)((uint32_t)(r0 >> 32) & code), (int)((uint32_t)(r1 >> 32) & code), (int)((uint32_t)(w >> 32) & code),
             (int)((uint32_t)(r3 >> 32) & code), 0, 0, 0, 0};
}

// cbsz = blgp = 4: both operands FP4 (E2M1); the E8M0 block scales of the operands are 2^0 (product = digit / 2 * 2).
__device__ __forceinline__ v4f mfma_fp4(const v8i a, const v8i b, const v4f c)
{
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 4, 4, 0, 127, 0, 127);
}

// NQ: chunks of 512 columns per wave; MAXS: most waves (column slices) per workgroup, which bounds
// the registers a wave may use; RU: units (row tile, bitlayer) whose blocks a wave has in flight.  The host picks
// RU <= the units a wave has, so that a short stream pays for no empty ring slots; 4 KB in flight per wave
// measured best (more requests in flight than that slow the short streams down and do not speed up the long ones).
template <int NQ, int MAXS, int RU>
__global__ __launch_bounds__(MAXS * 64) void k_mfma(const uint32_t *packed, const float *X0, uint32_t packed_bytes,
                                                    uint32_t flags, int cols0, uint32_t layer_step,
                                                    uint32_t round_step, int rounds_per_wg, int rt_count, int cq,
                                                    int m_used, const MfmaArgs a)
{
    const MfmaHead h = {packed, X0, packed_bytes, flags, cols0, layer_step, round_step, rounds_per_wg, rt_count, cq, m_used};
    // Units requested before the activations have arrived (a head start that keeps HBM busy during the transpose);
    // the rest of the ring follows once the digit rows are built.
    // (two units measured best: with three or four a call of 4096 or 8192 columns takes 0.2-0.5 us longer)
    constexpr int PRE = NQ >= 4 ? 1 : (RU < 2 ? RU : 2);
    // sums per bitlayer, row and kind of lane: the four operand rows of a lane of the result are
    // the even digits 0-6, the even digits 8-14, the odd digits 1-7, the odd digits 9-15.  The 64 lanes of a wave add to
    // different words.  Two buffers, used by alternate row tiles.
    __shared__ __align__(16) int abuf[2][PB_MAX_BITS][kTileRows][4];
    __shared__ float s_scales[PB_MAX_BITS];
    // staging area of the activation transpose, kStageRows rows of 8 bytes per wave (none when the planes are given)
    extern __shared__ __align__(16) unsigned char stage_lds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = (h.cq + NQ - 1) / NQ;                    // = blockDim.x / 64 (the launcher's S), from a preloaded argument
    const int m = h.m;
    const int rt0 = blockIdx.x * h.rounds_per_wg;
    const int rounds = min(h.rounds_per_wg, h.rt_count - rt0);  // >= 1 by construction
    int turn = 0;         // row tiles finished % nwaves, kept up by additions: the wave whose turn it is to finish a row tile
    const int q0 = wave * NQ;                                   // first chunk of this wave's column slice
    const int nq = min(NQ, h.cq - q0);                          // chunks it really has (>= 1 by construction)
    const int U = rounds * m;                                   // units: (row tile, bitlayer)

    // layer scales, lane i holds scales[i]: requested after the
    // first weights (nothing that a wave requests before them may depend on the argument structure, which is still
    // on its way when a wave starts); parked in LDS once the digit rows are built (the barrier before the first final
    // sum orders that store)
    // (Buffer loads whose range ends after m scales, none without scales: no branch, so that the compiler's count of
    // the loads in flight stays exact and a wait for the activations does not turn into a wait for the weights.)
    float scv = 0.0f;
    auto request_scales = [&]() {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(a.scales), 0, a.scales ? m * 4 : 0, 0x00020000);
        scv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, 0, 0));
    };

    // ---- the weight stream of this wave: unit u = (round r, bitlayer p): NQ blocks of 1 KB ----
    const size_t base_off = (size_t)rt0 * h.round_step + (size_t)q0 * 1024;
    const char *base = reinterpret_cast<const char *>(h.packed) + base_off;
    const uint32_t avail = (uint32_t)(h.packed_bytes - base_off);
    const int voff = lane * 16;
    // (non-temporal loads: a call reads every block once)
    constexpr int kWeightPolicy = 2;
    u32x4 ring[RU][NQ];
    uint32_t ld_round = 0;
    int ld_p = 0, ld_u = 0;
    auto issue = [&](u32x4 (&dst)[NQ]) {
        // past the last unit, and for chunks beyond the end of a ragged last slice, the descriptor has 0 records:
        // every lane is out of range, the load returns 0 and moves no data (no branch, so the compiler counts
        // the loads in flight exactly)
        const uint32_t off = ld_round + (uint32_t)ld_p * h.layer_step;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char *>(base), 0, (ld_u < U && q < nq) ? (int)avail : 0, 0x00020000);
            dst[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + q * 1024, (int)off, kWeightPolicy);
        }
        __builtin_amdgcn_sched_barrier(0x7);
        ++ld_u;
        if (++ld_p == m) { ld_p = 0; ld_round += h.round_step; }
    };

    // LDS sums start at zero.  The barrier that orders this is taken after every wave has REQUESTED its activations
    // and before any wave requests weights: the memory pipeline of a CU returns data in request order, so an
    // activation load queued behind another wave's weight loads (HBM misses) would arrive a memory latency late.
    auto zero_sums_and_meet = [&]() {
        for (int i = threadIdx.x; i < 2 * PB_MAX_BITS * 4 * kTileRows; i += nwaves * 64) (&abuf[0][0][0][0])[i] = 0;
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- the digit rows of this wave's slice, as A operands, kept in registers ----
    // lane l = 16 * kb + i: digit i (planes 2 i, 2 i + 1 of x_q) of the words 16 * q + 4 * kb + t
    const int kb = lane >> 4;
    u32x4 pa[NQ][4];
    if (h.flags & kPlanesGiven) {
        const uint32_t top = (lane & 15) == 15 ? 0x22222222u : 0u;
        uint4 pl0[NQ], pl1[NQ];
        const uint32_t *pl = a.planes + (2 * digit_of_row(lane & 15)) * (size_t)a.cwp + (size_t)q0 * 16 + 4 * kb;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            pl0[q] = pl1[q] = make_uint4(0, 0, 0, 0);
            if (q < nq) {
                pl0[q] = *reinterpret_cast<const uint4 *>(pl + q * 16);
                pl1[q] = *reinterpret_cast<const uint4 *>(pl + (size_t)a.cwp + q * 16);
            }
        }
        zero_sums_and_meet();
#pragma unroll
        for (int k = 0; k < PRE; ++k) issue(ring[k]);
        request_scales();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint4 p0 = pl0[q], p1 = pl1[q];
            digit_operand_from_planes(p0.x, p1.x, pa[q][0]);
            digit_operand_from_planes(p0.y, p1.y, pa[q][1]);
            digit_operand_from_planes(p0.z, p1.z, pa[q][2]);
            digit_operand_from_planes(p0.w, p1.w, pa[q][3]);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) pa[q][t][r] = signed_top_digit(pa[q][t][r], top);
        }
    } else {
        // Algorithm 2: x_q = Int(x * 2^f); then the transpose of Section 3.4 through LDS.  Lane L loads the
        // columns 256 j + 4 L .. + 3 (j = 0, 1) of a chunk with one 16-byte load each, converts them, writes the
        // sixteen digit codes of every column as one 8-byte row into this wave's staging area and reads the rows back
        // transposed: lane (kb, i) receives digit row i of the 32 columns of word 4 kb + t, register r = the
        // columns 4 n + r, which is the A operand as it stands.
        // Buffer loads return 0 beyond the end of the vector (checked dword by dword).
        uint2 *stage = reinterpret_cast<uint2 *>(stage_lds) + wave * kStageRows;
        uint2 *const wr_row = stage + stage_row(lane >> 3, 0, lane & 7);   // a load's four columns: word 8 j + (lane >> 3), n = lane & 7
        const uint2 *const rd_row = stage + stage_row(4 * kb, (lane >> 3) & 1, lane & 7);
        const int col0 = 512 * q0 + 4 * lane;                 // first column of the lane's load j = 0 of chunk 0
        u32x4 xv[NQ][2];
        {
            const __amdgpu_buffer_rsrc_t rx0 =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(h.X0), 0, h.cols0 * 4, 0x00020000);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    xv[q][j] = __builtin_amdgcn_raw_buffer_load_b128(rx0, (col0 + 512 * q + 256 * j) * 4, 0, 0);
        }
        // Second part of a concatenated input [X0 ; X1].  Offsets of columns that belong to the first part
        // would be negative: they are clamped and the value dropped (a negative register offset that an
        // instruction offset brings back above zero is not range-checked lane by lane on this hardware).
        // If cols0 is a multiple of 4, or the wave's slice begins beyond it, a lane's four columns lie in one part and one
        // 16-byte load serves; else every column is loaded by itself.
        u32x4 xw[NQ][2];
        if (h.flags & kSecondPart) {
            const __amdgpu_buffer_rsrc_t rx1 =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.X1), 0, a.cols1 * 4, 0x00020000);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int c1 = col0 + 512 * q + 256 * j - h.cols0;
                    if ((h.cols0 & 3) == 0 || 512 * q0 >= h.cols0) {
                        xw[q][j] = __builtin_amdgcn_raw_buffer_load_b128(rx1, max(c1, 0) * 4, 0, 0);
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            xw[q][j][r] = __builtin_amdgcn_raw_buffer_load_b32(rx1, max(c1 + r, 0) * 4, 0, 0);
                    }
                }
        }
        zero_sums_and_meet();
#pragma unroll
        for (int k = 0; k < PRE; ++k) issue(ring[k]);
        request_scales();
        if (h.flags & kSecondPart) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        xv[q][j][r] |= col0 + 512 * q + 256 * j + r >= h.cols0 ? xw[q][j][r] : 0u;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            // (the reads of the chunk before have returned: their registers were waited for below)
            // (32-bit activations need no clamp after the conversion: one instruction less per value)
            auto write_rows = [&](auto narrow) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        wr_row[stage_row(8 * j, r, 0)] = digit_codes((uint32_t)to_fixed_point<decltype(narrow)::value>(
                            __uint_as_float(xv[q][j][r]), a.fscale, a.imin, a.imax));
            };
            if (a.imin != INT32_MIN) write_rows(std::true_type{});
            else write_rows(std::false_type{});
            // the wave's own writes have landed before its lanes read each other's rows
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint2 lo = lds_read_transposed(rd_row + stage_row(t, 0, 0));
                const uint2 hi = lds_read_transposed(rd_row + stage_row(t, 2, 0));
                pa[q][t] = u32x4{lo.x, lo.y, hi.x, hi.y};
            }
            // ... and the reads have returned before the next chunk overwrites the rows
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (wave == 0 && lane < PB_MAX_BITS) s_scales[lane] = scv;
    __builtin_amdgcn_sched_barrier(0);   // the rest of the ring is requested after the activations have arrived
#pragma unroll
    for (int k = PRE; k < RU; ++k) issue(ring[k]);

    // The four registers of a lane of the result are the operand rows 4 kb + c: the digits b, b + 2, b + 4, b + 6
    // with b = 0, 8, 1, 9 for kb = 0 .. 3.  A lane adds them up with the weights 16^c (in units of 4^b) and the sums
    // of the four kinds of lanes stay apart until the row tile is finished.
    // Sums of digit products are <= 9 * 2048 (a slice has at most 2048 columns): c0 + 16 c1 and
    // c2 + 16 c3 are exact in fp32 (< 2^19), their combination is an integer below 2^27.
    const int j = lane & 15;
    int pp = 0, pr = 0;   // bitlayer and round of the unit being multiplied
    for (int u0 = 0; u0 < U; u0 += RU) {
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            if (u0 + k < U) {
                // (chunks beyond a ragged last slice are zero words)
                v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const u32x4 w = ring[k][q];
#pragma unroll
                    for (int t = 0; t < 4; t += 2) {
                        v8i b0, b1;
                        weight_operands((uint64_t)w[t + 1] << 32 | w[t], b0, b1);
                        acc = mfma_fp4(as_operand(pa[q][t]), b0, acc);
                        acc = mfma_fp4(as_operand(pa[q][t + 1]), b1, acc);
                    }
                }
                // the end of a bitlayer: the sum of this lane goes to its set in LDS
                {
                    const float t0 = fmaf(acc[1], 16.0f, acc[0]), t1 = fmaf(acc[3], 16.0f, acc[2]);
                    atomicAdd(&abuf[pr & 1][pp][j][kb], (int)t0 + ((int)t1 << 8));
                }
                if (++pp == m) {
                    // The row tile is complete in every slice: scale and store it.  (The barrier per row tile also
                    // keeps the waves of a workgroup on one contiguous region of the weight stream; letting them
                    // drift apart over several row tiles measured 5-15 % slower.)
                    // Four lanes per row share out the
                    // bitlayers: scaled sums in fp64, then the sum over those lanes (16 and 32 lanes apart).
                    // The waves take turns, so that none of them is always late for the next barrier.
                    pp = 0;
                    __syncthreads();
                    if (wave == turn) {
                        const int lg = kb, jrow = j;
                        const int prow = (rt0 + pr) * kTileRows + jrow;
                        const int row = a.gate_h ? gates_matrix_row(prow, a.gate_h) : prow;
                        const bool row_ok = row >= 0 && row < a.R;
                        int4 *src = reinterpret_cast<int4 *>(&abuf[pr & 1][lg][jrow][0]);
                        // bias and previous cell state of this lane's outputs: requested before the sums are read and
                        // added up, so that their way through memory is not waited for at the end (range-checked
                        // loads: 0 for absent arrays and for lanes without an output)
                        constexpr int kNoOutput = 0x7FFFFFF0;   // an offset beyond every array
                        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<float *>(a.bias), 0, a.bias ? a.R * 4 : 0, 0x00020000);
                        const float bias_row =
                            __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, row_ok ? row * 4 : kNoOutput, 0, 0));
                        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<float *>(a.c_prev), 0, a.c_prev ? a.gate_h * 4 : 0, 0x00020000);
                        const bool cell = row_ok && (lane & 3) == 0;
                        const float c_old =
                            __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, cell ? row * 4 : kNoOutput, 0, 0));
                        double z = 0.0;
                        // the quarters of the vector: digits 0, 2, 4, 6 in units of 1, digits 8 .. 14 in units
                        // of 4^8, digits 1 .. 7 in units of 4, digits 9 .. 15 in units of 4^9; each below 2^31 in
                        // magnitude (4369 * 9 * 32768 columns)
                        constexpr int SET = kTileRows;   // int4s from one set of sums to the next
                        if (a.A) {
                            for (int i = lg; i < m; i += 4, src += 4 * SET) {
                                const int4 t = *src;
                                *src = make_int4(0, 0, 0, 0);
                                const long long sum = (long long)t.x + 4 * (long long)t.z + (((long long)t.y + 4 * (long long)t.w) << 16);
                                if (row_ok) a.A[(size_t)i * (size_t)a.R + row] = sum;
                            }
                        } else {
                            // The sets of a lane are read CH at a time, together with their scales, so that the LDS
                            // latency is paid once: sets beyond the last one hold zeros (nothing ever adds to them) and
                            // add nothing.  The 32-bit parts convert to fp64 exactly and so does their combination
                            // (below 2^51), which is the integer sum itself.
                            constexpr int MAXI = PB_MAX_BITS / 4;   // sets a lane can have
                            constexpr int CH = 2;                   // (a chunk covers eight sets)
                            static_assert(MAXI % CH == 0, "whole chunks");
                            for (int k0 = 0; k0 * 4 < m; k0 += CH, src += CH * 4 * SET) {
                                int4 t[CH];
                                float sc[CH];
#pragma unroll
                                for (int c = 0; c < CH; ++c) {
                                    t[c] = src[c * 4 * SET];
                                    sc[c] = s_scales[lg + 4 * (k0 + c)];   // (below PB_MAX_BITS)
                                }
#pragma unroll
                                for (int c = 0; c < CH; ++c) src[c * 4 * SET] = make_int4(0, 0, 0, 0);
#pragma unroll
                                for (int c = 0; c < CH; ++c) {
                                    const double sum = fma(65536.0, fma(4.0, (double)t[c].w, (double)t[c].y),
                                                           fma(4.0, (double)t[c].z, (double)t[c].x));
                                    z = fma((double)sc[c], sum, z);
                                }
                            }
                        }
                        z = add_across<16>(z);
                        z = add_across<32>(z);
                        if (!a.A) {
                            float y = (float)(z * a.out_scale);
                            if (a.bias && row_ok) y += bias_row;
                            if (a.c_prev) {
                                // LSTM cell: the four lanes of a quad hold the gates i, f, g, o of one unit (row =
                                // unit for gate i)
                                float cn, hn;
                                lstm_quad(y, lane, c_old, &cn, &hn);
                                if (cell && lg == 0) {
                                    a.c_out[row] = cn;
                                    a.h_out[row] = hn;
                                }
                            } else {
                                if (a.relu) y = fmaxf(y, 0.0f);
                                if (row_ok && lg == 0) a.Y[row] = y;
                            }
                        }
                    }
                    ++pr;
                    if (++turn == nwaves) turn = 0;
                }
            }
            issue(ring[k]);
        }
    }
}

// The kernel variants: (chunks per wave, most slices per workgroup, ring depth in units)
struct Variant {
    int nq, maxs, ru;
    const void *fn;
};
#define PB_VARIANT(NQ, MAXS, RU) {NQ, MAXS, RU, reinterpret_cast<const void *>(k_mfma<NQ, MAXS, RU>)}
static const Variant kVariants[] = {
    PB_VARIANT(1, 16, 1), PB_VARIANT(1, 16, 2), PB_VARIANT(1, 16, 4),
    PB_VARIANT(2, 16, 1), PB_VARIANT(2, 16, 2), PB_VARIANT(2, 16, 3),
    PB_VARIANT(4, 8, 1),  PB_VARIANT(4, 8, 2),
    PB_VARIANT(4, 16, 1),
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

// Overrides of the launcher's choices (chunks per wave, ring depth, workgroups), for sweeps over
// the variants: compiled in only with -DPB_TUNING (a tuning build reads them from the environment once); the
// product build has none and its behaviour does not depend on the environment.  0 = not set.
struct Tuning {
    int nq = 0, ru = 0, wgs = 0;
#ifdef PB_TUNING
    Tuning()
    {
        auto get = [](const char *name) { const char *e = getenv(name); return e && atoi(e) > 0 ? atoi(e) : 0; };
        nq = get("PB_TUNE_NQ"); ru = get("PB_TUNE_RU"); wgs = get("PB_TUNE_WGS");
    }
#endif
};
static const Tuning &tuning()
{
    static const Tuning t;
    return t;
}

// The smallest slice (most waves per row, shortest transpose per wave) whose slice
// count fits a workgroup; ring depth 1 (the deeper rings are picked once the units per wave are known).
static int pick_variant(const Layout &L)
{
    int best = -1;
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        if (v.ru != 1 || (L.cq + v.nq - 1) / v.nq > v.maxs) continue;
        if (tuning().nq && v.nq != tuning().nq) continue;
        if (best < 0 || v.nq < kVariants[best].nq) best = i;
    }
    return best;
}

// The sibling of variant `vi` with the deepest ring that a wave with `units` units fills; with three units and
// rings of 2 and 4 to choose from, the deeper one (a wave with one or two units is faster without empty ring slots,
// one with three is 0.2 us faster when all three are in flight).
static int pick_ring(int vi, int units)
{
    const int want = tuning().ru, cap = units == 3 ? 4 : units;
    int best = vi;
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        if (v.nq != kVariants[vi].nq || v.maxs != kVariants[vi].maxs) continue;
        if (want ? v.ru == want : (v.ru <= cap && v.ru > kVariants[best].ru)) best = i;
    }
    return best;
}

// Dynamic LDS of a workgroup of S waves: the staging area of the activation transpose.
static size_t stage_bytes(int S) { return (size_t)S * kStageRows * sizeof(uint2); }

// Workgroups of S waves that fit on the device at once (occupancy does not change while the process lives, so it
// is looked up once per kernel variant and workgroup size).
static int resident_workgroups(int variant, int S)
{
    static int cache[kNumVariants][kMaxSlices + 1];
    int *slot = &cache[variant][S];
    int v = __atomic_load_n(slot, __ATOMIC_RELAXED);
    if (v > 0) return v;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    // (a workgroup's dynamic LDS may exceed the default limit of 64 KB, a compute unit of this chip has 160 KB:
    // declared for this variant and its siblings of other ring depths, one of which is the one launched)
    if (stage_bytes(S) > 32 * 1024) {
        for (int i = 0; i < kNumVariants; ++i) {
            const Variant &o = kVariants[i];
            if (o.nq != kVariants[variant].nq || o.maxs != kVariants[variant].maxs) continue;
            if (hipFuncSetAttribute(o.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)stage_bytes(S)) != hipSuccess)
                return 0;
        }
    }
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kVariants[variant].fn, S * 64, stage_bytes(S)) != hipSuccess)
        return 0;
    v = cus * per_cu;
    if (v > 0) __atomic_store_n(slot, v, __ATOMIC_RELAXED);
    return v;
}

int launch_mfma(const uint32_t *packed, const float *scales, const Layout &L, int bits_used, int frac_bits,
                int act_bits, const float *X0, int cols0, const float *X1, int cols1, const uint32_t *planes, float *Y,
                long long *A, const Epilogue &ep, hipStream_t st)
{
    MfmaArgs a;
    MfmaHead h;
    h.packed = packed; h.X0 = X0; a.X1 = X1; a.planes = planes; a.scales = scales; a.Y = Y; a.A = A;
    a.bias = ep.bias; a.relu = ep.relu; a.c_prev = ep.c_prev; a.h_out = ep.h_out; a.c_out = ep.c_out;
    a.gate_h = L.gate_h;
    // (the epilogue addresses the bias and the cell state with 32-bit byte offsets)
    if (ep.bias && L.rows >= (1 << 29)) return (int)hipErrorInvalidValue;
    if (ep.c_prev && L.gate_h >= (1 << 29)) return (int)hipErrorInvalidValue;
    h.packed_bytes = (uint32_t)packed_bytes(L);   // (the host API refuses matrices of 4 GiB and more)
    h.flags = (planes ? kPlanesGiven : 0u) | (X1 ? kSecondPart : 0u);
    h.layer_step = (uint32_t)(tile16_layer_stride(L) * 4);
    h.round_step = (uint32_t)(tile16_rowtile_stride(L) * 4);
    h.cols0 = cols0; a.cols1 = cols1;
    a.R = L.rows; h.rt_count = L.rt_count; h.cq = L.cq; a.cwp = L.cwp;
    h.m = bits_used;
    a.fscale = ldexpf(1.0f, frac_bits);
    a.imax = (act_bits == 32) ? INT32_MAX : (int32_t)((1u << (act_bits - 1)) - 1u);
    a.imin = -a.imax - 1;
    a.out_scale = ldexp(1.0, -frac_bits);
    const int vi = pick_variant(L);
    if (vi < 0) return (int)hipErrorInvalidValue;
    const Variant &var = kVariants[vi];   // (the ring depth does not change a variant's occupancy: same registers +- a few)
    const int S = (L.cq + var.nq - 1) / var.nq;
    // Workgroups: as many as are resident at once (so that every wave builds its planes once and the weight
    // stream never waits for a second round of workgroups to start), each with whole row tiles.
    int wgs = resident_workgroups(pick_ring(vi, 1 << 30), S);   // of the sibling that needs the most registers
    if (wgs < 1) return (int)hipErrorInvalidValue;
    if (tuning().wgs > 0) wgs = tuning().wgs;
    if (wgs > L.rt_count) wgs = L.rt_count;
    h.rounds_per_wg = (L.rt_count + wgs - 1) / wgs;
    wgs = (L.rt_count + h.rounds_per_wg - 1) / h.rounds_per_wg;
    const Variant &run = kVariants[pick_ring(vi, h.rounds_per_wg * bits_used)];
    void *args[] = {&h.packed, &h.X0, &h.packed_bytes, &h.flags, &h.cols0, &h.layer_step, &h.round_step,
                    &h.rounds_per_wg, &h.rt_count, &h.cq, &h.m, &a};
    const hipError_t e = hipLaunchKernel(run.fn, dim3((unsigned)wgs), dim3((unsigned)S * 64), args,
                                         planes ? 0 : stage_bytes(S), st);
    return (int)(e != hipSuccess ? e : hipGetLastError());
}

}  // namespace pb
