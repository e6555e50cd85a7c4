// Internal: what the two product kernels on the 8-bit integer matrix cores share (pb_imma.hip, pb_imma_tile.hip).
//
// The product of Algorithm 2 as whole weight codes times the bytes of the fixed-point activations on the 8-bit integer
// matrix cores.
//
// The bitlayers of a weight matrix with the scales of Algorithm 1 (each half the one before, the sign bitlayer minus
// twice its neighbour) are the two's-complement bits of one integer code, so
//     sum_i scales[i] A_i = scales[last] * sum_c code[c] x_q[c]
// and up to eight bitlayers are multiplied at once: eight packed words become the codes of 32 columns (a transpose of
// 8 x 8 bits, 40 operations of the vector ALU) and V_MFMA_I32_16X16X64_I8 multiplies them with the bytes of x_q.
// A 32-bit x_q is four byte digits: against the sixteen base-4 digits and bitlayer pairs of the FP4 form that is 4
// products per weight and activation instead of 64, at half the rate per product.
//
// Digits.  The top byte of x_q is signed as it stands; a lower byte u enters as s = u - 128 (u ^ 0x80 read as signed), so
//     x_q = sum_d 256^d s_d + K,   K = 0x808080 (four bytes), 0x80 (two), 0 (one),
// and K * sum_c code[c] is added per weight row: one more matrix instruction per weight operand, with an operand of
// ones, delivers that sum.  |s_d code| <= 2^14, so a sum over all 32768 columns stays below 2^30: int32 is exact.
// Three of four: a 32-bit x_q in [-2^23, 2^23) is the sum of its lower three bytes with the third one signed as it stands and
// K = 0x8080.  k_digits leaves the third byte as it stands and notes for four vectors and a chunk of columns whether a value is
// wider.  Where none is, the top digits are not read (and not multiplied, in k_i8_tile); else the product kernel turns the third digit
// to u ^ 0x80.  Where k_i8 with one tile of digit rows follows, mostly all four digits are used and k_digits turns the third.
//
// Groups.  A group of bitlayers [f, e) is one code: bitlayer i stands at slot i (counted from bit 7 down) in the first
// group, which may hold eight, and at slot i - f + 2 in the later ones, which hold up to six (the sign bit and the one
// below it stay clear).  Scales that do not halve are groups of one bitlayer each; so are the sums that pb_matmul_acc asks for,
// and groups of two those of pb_matmul_acc_pairs.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pb_device.h"
#include "pb_kernels.h"

namespace pb {

typedef int v4i __attribute__((ext_vector_type(4)));

// Where the activations come from: row n = [X0[n][0..cols0) ; X1[n][0..cols1)], fp32.
struct ActSource {
    const float *X0, *X1;
    int cols0, cols1;
    int batch;
    float fscale;       // 2^frac_bits
    int imin, imax;     // range of the act_bits-bit fixed-point values
};

// An offset beyond every buffer: a load there returns 0 (buffer loads are range-checked lane by lane)
constexpr int kNowhere = 0x7FFFFFF0;

// The columns c + 8 b + r (b, r = 0..3; c a multiple of 4) of vector n as they are in memory; 0 beyond the ends.
// `end` (the same in all lanes) is beyond every column that the wave asks for, all of which lie in the 512 before it.
__device__ __forceinline__ void load_columns(const ActSource &s, int n, int c, int end, u32x4 (&v)[4])
{
    const bool live = n < s.batch;
    const __amdgpu_buffer_rsrc_t r0 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(s.X0), 0, (int)((uint32_t)s.batch * (uint32_t)s.cols0 * 4u), 0x00020000);
    const int off = (n * s.cols0 + c) * 4;
#pragma unroll
    for (int b = 0; b < 4; ++b)
        v[b] = __builtin_amdgcn_raw_buffer_load_b128(r0, live && c + 8 * b < s.cols0 ? off + 32 * b : kNowhere, 0, 0);
    if ((s.cols0 & 3) && end > s.cols0) {   // (four columns that reach into the next row)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[b][r] = c + 8 * b + r < s.cols0 ? v[b][r] : 0u;
    }
    if (s.X1 && end > s.cols0) {
        const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(s.X1), 0, (int)((uint32_t)s.batch * (uint32_t)s.cols1 * 4u), 0x00020000);
        const int c1 = c - s.cols0, off1 = (n * s.cols1 + c1) * 4;
        // (all requests before the first value is used, and three single values where the parts meet in place of sixteen: a step of an LSTM cell
        // of 279 units and 75 inputs, 35 vectors of 8 bits, 14.5 -> 12.0 us; 177 units and 87 inputs, 3 vectors of 16 bits, 6.5 -> 6.1)
        u32x4 w[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int cb = c1 + 8 * b;
            w[b] = __builtin_amdgcn_raw_buffer_load_b128(r1, live && cb >= 0 && cb < s.cols1 ? off1 + 32 * b : kNowhere, 0, 0);
        }
        const int lead = s.cols0 & 3;
        uint32_t e[4] = {};
        if (lead != 0 && end - 512 < s.cols0) {   // the four columns in which the second part begins: up to three of its values
#pragma unroll
            for (int r = 1; r < 4; ++r) {
                const int x = r - lead;
                e[r] = __builtin_amdgcn_raw_buffer_load_b32(r1, live && x >= 0 && x < s.cols1 ? (n * s.cols1 + x) * 4 : kNowhere, 0, 0);
            }
        }
        const int b0 = s.cols0 - lead - c;        // (8 b: they are v[b])
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[b][r] |= c1 + 8 * b + r < s.cols1 ? w[b][r] : 0u;
                if (r > 0) v[b][r] |= b0 == 8 * b ? e[r] : 0u;
            }
    }
}

__device__ __forceinline__ void convert_columns(const ActSource &s, u32x4 (&v)[4])
{
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[b][r] = (uint32_t)to_fixed_point<true>(__uint_as_float(v[b][r]), s.fscale, s.imin, s.imax);
}

// Sixteen fixed-point values, v[b][r] = column 8 b + r, -> their byte digits: word r of out[d] holds digit d of the columns r,
// 8 + r, 16 + r, 24 + r, the order in which weight_codes() leaves the codes of 32 columns. 
template <int ND>
__device__ __forceinline__ void byte_digits(const u32x4 (&v)[4], u32x4 (&out)[ND])
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (ND == 1) {
            const uint32_t a = __builtin_amdgcn_perm(v[1][r], v[0][r], 0x0C0C0400u);
            const uint32_t b = __builtin_amdgcn_perm(v[3][r], v[2][r], 0x0C0C0400u);
            out[0][r] = __builtin_amdgcn_perm(b, a, 0x05040100u);
        } else {
            const uint32_t a = __builtin_amdgcn_perm(v[1][r], v[0][r], 0x05010400u);
            const uint32_t b = __builtin_amdgcn_perm(v[3][r], v[2][r], 0x05010400u);
            out[0][r] = __builtin_amdgcn_perm(b, a, 0x05040100u) ^ 0x80808080u;
            out[1][r] = __builtin_amdgcn_perm(b, a, 0x07060302u);
            if constexpr (ND == 4) {
                out[1][r] ^= 0x80808080u;
                const uint32_t c = __builtin_amdgcn_perm(v[1][r], v[0][r], 0x07030602u);
                const uint32_t d = __builtin_amdgcn_perm(v[3][r], v[2][r], 0x07030602u);
                out[2][r] = __builtin_amdgcn_perm(d, c, 0x05040100u) ^ 0x80808080u;
                out[3][r] = __builtin_amdgcn_perm(d, c, 0x07060302u);
            }
        }
    }
}

// 130 cycles a word instead of 220 with V_BFI_B32 and shifts of 32 bits (see pb_device.h); of a kernel's time, where the codes are only a
// part of it: 1500 x 700, 4 bitlayers, 30 vectors of 16 bits 5.84 -> 5.53 us, 2002 x 5817, one bitlayer, 2 vectors 5.33 -> 4.98, 67 x 6211,
// 16 bitlayers, 3 vectors 11.6 -> 10.7, 8192 x 8192, 4 vectors 14.05 -> 13.9.
struct Masks { uint32_t m1, m2, m4; };   // 0xAA.., 0xCC.., 0xF0..
__device__ __forceinline__ Masks make_masks() { return {in_vgpr(0xAAAAAAAAu), in_vgpr(0xCCCCCCCCu), in_vgpr(0xF0F0F0F0u)}; }
__device__ __forceinline__ uint32_t twice(uint32_t v)
{
    uint32_t r;
    asm("v_add_u32 %0, %1, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ uint64_t both(uint32_t a, uint32_t b) { return (uint64_t)b << 32 | a; }
// (a & mask) | (b & ~mask)
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA); }
__device__ __forceinline__ uint64_t mix(uint32_t mask, uint64_t a, uint64_t b)
{
    return both(pick(mask, (uint32_t)a, (uint32_t)b), pick(mask, (uint32_t)(a >> 32), (uint32_t)(b >> 32)));
}

// Two words by N, together or each by itself: the kernel with four tiles of digit rows per wave is faster with the latter (8192 x 8192, 16
// vectors 24.5 us, together 26.4, V_BFI_B32 24.6; over 216 drawn calls 5.4 % on average), all others with the former.
template <int N, bool SHIFT64>
__device__ __forceinline__ uint64_t shifted_up(uint64_t v)
{
    return SHIFT64 ? up<N>(v) : both((uint32_t)v << N, (uint32_t)(v >> 32) << N);
}
template <int N, bool SHIFT64>
__device__ __forceinline__ uint64_t shifted_down(uint64_t v)
{
    return SHIFT64 ? down<N>(v) : both((uint32_t)v >> N, (uint32_t)(v >> 32) >> N);
}

// Four words of adjacent slots (p[0] the highest bit) -> four words of 4-bit codes, v[0] = (k = 0, k = 1), v[1] = (k = 2, k = 3): nibble n
// of word k holds the bits p[0][c] p[1][c] p[2][c] p[3][c] of column c = 4 n + k.  IL: (p[0], p[1]) and (p[2], p[3]) are the even and the
// odd columns' digits of a bitlayer pair already, one exchange less.
template <bool IL, bool SHIFT64>
__device__ __forceinline__ void nibble_codes(const Masks &m, const uint32_t *p, uint64_t (&v)[2])
{
    uint64_t h, l;   // (even columns, odd columns) of the upper and of the lower two slots
    if constexpr (IL) {
        h = both(p[0], p[1]);
        l = both(p[2], p[3]);
    } else {
        h = both(pick(m.m1, twice(p[0]), p[1]), pick(m.m1, p[0], p[1] >> 1));
        l = both(pick(m.m1, twice(p[2]), p[3]), pick(m.m1, p[2], p[3] >> 1));
    }
    v[0] = mix(m.m2, shifted_up<2, SHIFT64>(h), l);
    v[1] = mix(m.m2, h, shifted_down<2, SHIFT64>(l));
}

// The words of 4 Q slots (slot 0 = bit 7) of 32 columns -> their codes: byte b of lo[k] is the code of column 8 b + k, byte b of
// hi[k] that of column 8 b + 4 + k
template <int Q, bool IL, bool SHIFT64>
__device__ __forceinline__ void weight_codes(const Masks &m, const uint32_t (&w)[4 * Q], v4i &lo, v4i &hi)
{
    uint64_t a[2], b[2] = {};
    nibble_codes<IL, SHIFT64>(m, w, a);
    if constexpr (Q == 2) nibble_codes<IL, SHIFT64>(m, w + 4, b);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint64_t l = mix(m.m4, shifted_up<4, SHIFT64>(a[k]), b[k]);
        const uint64_t h = mix(m.m4, a[k], Q == 2 ? shifted_down<4, SHIFT64>(b[k]) : 0);
        lo[2 * k] = (int)(uint32_t)l;
        lo[2 * k + 1] = (int)(l >> 32);
        hi[2 * k] = (int)(uint32_t)h;
        hi[2 * k + 1] = (int)(h >> 32);
    }
}
// Word t of the slots' pieces.  IL: the sign bitlayer is stored complemented (`flip`), and a pair may hold a bit that does
// not belong to the group (`mask`)
template <int Q, bool IL>
__device__ __forceinline__ void words_of(const u32x4 (&w)[4 * Q], int t, uint32_t flip, const uint32_t (&mask)[2 * Q], uint32_t (&p)[4 * Q])
{
#pragma unroll
    for (int s = 0; s < 4 * Q; ++s) {
        p[s] = w[s][t];
        if constexpr (IL) p[s] = (s < 2 ? p[s] ^ flip : p[s]) & mask[s / 2];
    }
}

// The byte digits in memory: [group of 16 vectors][chunk of 512 columns][t = word % 4][h][quad of vectors][digit][kb = word / 4][vector of
// the quad][16 bytes], the 16 bytes being the columns 8 b + 4 h + r of the word; a last quad of fewer vectors has as many fewer bytes
// per kb.  An operand of four vectors' four digits is 1 KB in one piece, one of a digit of sixteen vectors is four pieces of 256 bytes.
// Beside them, for 32-bit values, a byte per quad (64 apart) and chunk: 1 if a value is outside [-2^23, 2^23).
constexpr int kGroupVectors = 16;
__host__ __device__ inline int group_vectors(int batch, int group)
{
    const int left = batch - group * kGroupVectors;
    return left < 0 ? 0 : (left < kGroupVectors ? left : kGroupVectors);
}
// From one (t, h) to the next, and the sixteen bytes of (digit, kb, vector v of the group) in the first one
__device__ __forceinline__ uint32_t digits_step(int vectors, int nd) { return (uint32_t)(vectors * nd * 64); }
__device__ __forceinline__ uint32_t digits_at(int group, int vectors, int cq, int nd, int digit, int kb, int v)
{
    const int quad = v & ~3, in_quad = vectors - quad < 4 ? vectors - quad : 4;
    return (uint32_t)group * (uint32_t)(kGroupVectors * 512 * nd) * (uint32_t)cq +
           (uint32_t)(quad * nd * 64 + ((digit * 4 + kb) * in_quad + (v & 3)) * 16);
}

struct I8Args {
    const uint32_t *packed;
    uint32_t packed_bytes;               // (below 2^32)
    uint32_t layer_step, round_step;     // bytes from one bitlayer of a row tile to the next, from one row tile to the next
    int rounds_per_wg;                   // row tiles per workgroup
    int rt_count, cq;
    int m;                               // bitlayers to accumulate
    int chunks_per_wave, stage_rows;     // (k_i8) chunks of 512 columns per wave, digit rows staged per tile
    const uint8_t *digits;               // prepared byte digits (not FUSED)
    uint32_t digits_bytes;
    ActSource act;
    const float *scales;
    float *Y;
    long long *A;
    int pairs_out;
    const float *bias;
    const float *c_prev;
    float *h_out, *c_out;
    int relu;
    int gate_h;
    int R;
    double out_scale;
    const uint8_t *wide;                 // beside the digits
};

// What a kernel does with the sums: store Y (bias and ReLU first), update the LSTM cell, store the sums themselves
enum { kStore = 0, kCell = 1, kSums = 2 };

// Whether one of the values of so many quads of vectors needs four digits (the lanes see one chunk each: there are at most 64)
template <int QUADS>
__device__ __forceinline__ uint32_t load_wide(const I8Args &a, int quad, int lane)
{
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.wide), 0, (a.act.batch + 3) / 4 * 64, 0x00020000);
    uint32_t v = 0;
#pragma unroll
    for (int i = 0; i < QUADS; ++i)
        v |= __builtin_amdgcn_raw_buffer_load_b8(rw, lane < a.cq ? (quad + i) * 64 + lane : kNowhere, 0, 0);
    return v;
}
__device__ __forceinline__ bool is_wide(uint32_t loaded) { return __builtin_amdgcn_ballot_w64(loaded != 0) != 0; }

// A group of bitlayers [f, e): its last bitlayer stands at `slot`, its sum counts `scale`
struct Group { int f, e, slot; bool first, last; double scale; };
__device__ __forceinline__ Group make_group(const I8Args &a, int f, int e, const float *scales)
{
    Group g;
    g.f = f; g.e = e;
    g.slot = e - 1 - ((f & ~1) == 0 ? 0 : (f & ~1) - 2);
    g.first = f == 0;
    g.last = e == a.m;
    g.scale = 0.0;
    if (!a.A) {
        const double s = (double)scales[e - 1];
        g.scale = ldexp(g.slot == 0 ? -s : s, g.slot - 7);
    }
    return g;
}

// The bias of packed row `prow` (0 without one)
__device__ __forceinline__ float bias_of(const I8Args &a, int prow)
{
    const int row = a.gate_h ? gates_matrix_row(prow, a.gate_h) : prow;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.bias), 0, a.R * 4, 0x00020000);
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, row >= 0 && row < a.R ? row * 4 : kNowhere, 0, 0));
}

// The sum of one vector and weight row from its digits' sums d[0 .. nd) and the sum of the row's codes, times the scale of the
// group (every part is an integer below 2^53 and exact; the last step rounds once if the sum is beyond).  The sum over the groups
// starts at +0: no zero with the sign of a scale.  `wide`: (four digits) the third one was turned to u ^ 0x80.
template <int ND>
__device__ __forceinline__ double scaled_sum(const Group &g, const int *d, int sum1, bool wide)
{
    double v = (double)d[0];
    if constexpr (ND == 2) v = fma(256.0, (double)d[1], fma(128.0, (double)sum1, v));
    if constexpr (ND == 4) {
        v = fma(65536.0, (double)d[2], fma(256.0, (double)d[1], v));
        v = fma(16777216.0, (double)d[3], fma(wide ? 8421504.0 : 32896.0, (double)sum1, v));
    }
    return fma(v, g.scale, 0.0);
}
template <int ND>
__device__ __forceinline__ long long integer_sum(const Group &g, const int *d, int sum1, bool wide)
{
    long long v = (long long)d[0];
    if constexpr (ND == 2) v += ((long long)d[1] << 8) + 0x80ll * sum1;
    if constexpr (ND == 4)
        v += ((long long)d[1] << 8) + ((long long)d[2] << 16) + ((long long)d[3] << 24) + (wide ? 0x808080ll : 0x8080ll) * sum1;
    v >>= 7 - g.slot;
    return g.slot == 0 ? -v : v;   // (the sign bitlayer by itself)
}

// The previous cell state of vector n and the unit of this lane's quad (0 in the lanes that do not update it)
__device__ __forceinline__ float cell_state(const I8Args &a, int lane, int row, bool row_ok, int n)
{
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.c_prev), 0,
                                                                        a.act.batch * a.gate_h * 4, 0x00020000);
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
        rc, row_ok && n < a.act.batch && (lane & 3) == 0 ? (n * a.gate_h + row) * 4 : kNowhere, 0, 0));
}

// What follows the product for vector n and matrix row `row` of this lane: v = its scaled sum over the groups up to this one
template <int EPI>
__device__ __forceinline__ void finish(const I8Args &a, int lane, int row, bool row_ok, int n, double v, float bias_row,
                                       float c_old)
{
    const bool live = row_ok && n < a.act.batch;
    float y = (float)(v * a.out_scale);
    if (a.bias) y += bias_row;
    if constexpr (EPI == kCell) {
        float cn, hn;
        lstm_quad(y, lane, c_old, &cn, &hn);
        if ((lane & 3) == 0 && live) {
            const size_t at = (size_t)n * a.gate_h + (size_t)row;
            a.c_out[at] = cn;
            a.h_out[at] = hn;
        }
    } else {
        if (a.relu) y = fmaxf(y, 0.0f);
        if (live) a.Y[(size_t)n * a.R + row] = y;
    }
}
__device__ __forceinline__ void store_sum(const I8Args &a, const Group &g, int row, bool row_ok, int n, long long v)
{
    if (row_ok && n < a.act.batch)
        a.A[((size_t)(a.pairs_out ? g.f / 2 : g.f) * a.act.batch + n) * (size_t)a.R + row] = v;
}

// Groups of bitlayers of a call that accumulates m of them with the scales of Algorithm 1 (at most four slots: one quad of words)
inline int i8_groups(int m)
{
    const int first = m <= 4 ? 4 : 8, later = first - 2;
    return m <= first ? 1 : 1 + (m - first + later - 1) / later;
}

// The kernel for many digit rows (pb_imma_tile.hip): its shapes (waves along the digit rows and as many column slots, tiles of
// sixteen digit rows per wave), the row tiles that a workgroup does, its launch
struct TileShape { int nt, tm; };
constexpr int kTileShapes = 3;
constexpr TileShape kTile[kTileShapes] = {{4, 2}, {8, 2}, {8, 4}};
inline int tile_rows(const TileShape &t, int m, bool sums)
{
    const int groups = sums ? t.nt : i8_groups(m);
    return groups >= t.nt ? 1 : t.nt / groups;
}
int launch_imma_tile(int shape, const I8Args &a, int nd, bool il, hipStream_t st);

}  // namespace pb
