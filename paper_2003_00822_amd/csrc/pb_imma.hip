// The product of Algorithm 2 for batches, and for the layout that stores bitlayer pairs, on the 8-bit integer matrix cores
// (see pb_imma.h for the arithmetic): the activations as byte digits, the kernel for few digit rows, and the choice
// between it and the kernel for many.
#include <stdlib.h>

#include "pb_imma.h"

namespace pb {

// The activations as byte digits in memory, for the calls that read them more than once (pb_imma.h has the order).
// A workgroup does one chunk of four vectors, each of its two waves the words t, t + 1 (mod 4).  The lanes are in the order in which the
// digits lie in memory: the order of the activations, two lanes to a word, took 0.2 us longer (56 vectors, 1402 columns).
// `turn`: what makes u of the third byte's u ^ 0x80.
template <int ND>
__global__ __launch_bounds__(128) void k_digits(ActSource s, int cq, uint8_t *__restrict__ digits, uint8_t *__restrict__ wide,
                                                int32_t *__restrict__ xq_out, const uint32_t turn)
{
    __shared__ int s_wide[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = blockIdx.x, quad = blockIdx.y, group = quad * 4 / kGroupVectors;
    const int kb = (lane >> 2) & 3, th = 4 * wave + (lane >> 4), n = 4 * quad + (lane & 3);
    const int vec = n % kGroupVectors, vectors = group_vectors(s.batch, group);
    const int c = 512 * q + 32 * (4 * kb + th / 2) + 4 * (th % 2);
    u32x4 v[4];
    load_columns(s, n, c, 512 * (q + 1), v);
    convert_columns(s, v);
    if (xq_out && n < s.batch) {
        const int cols = s.cols0 + s.cols1;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (c + 8 * b + r < cols) xq_out[(size_t)n * cols + c + 8 * b + r] = (int32_t)v[b][r];
    }
    u32x4 out[ND];
    byte_digits<ND>(v, out);
    if constexpr (ND == 4) out[2] ^= turn;
    if (vec < vectors) {
        uint8_t *dst = digits + (size_t)(q * 8 + th) * digits_step(vectors, ND);
#pragma unroll
        for (int d = 0; d < ND; ++d) *reinterpret_cast<u32x4 *>(dst + digits_at(group, vectors, cq, ND, d, kb, vec)) = out[d];
    }
    if constexpr (ND == 4) {
        uint32_t high = 0;   // bits that differ from the sign
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) high |= v[b][r] ^ (uint32_t)((int32_t)v[b][r] >> 31);
        const bool any = __builtin_amdgcn_ballot_w64(high >> 23 != 0) != 0;
        if (lane == 0) s_wide[wave] = any;
        __syncthreads();
        if (threadIdx.x == 0) wide[quad * 64 + q] = (uint8_t)(s_wide[0] | s_wide[1]);
    }
}

// ---------------------------------------------------------------------------------------------------------------

// Waves of a workgroup at most: sixteen have 128 registers each, which four tiles of digit rows exceed
__host__ __device__ constexpr int stream_waves(int tm) { return tm >= 4 ? 8 : 16; }

// LDS of a workgroup beside the staged digits: sums, sums of the codes, sums over the groups, scales
__host__ __device__ constexpr int stream_lds(int nd, int tm, int epi)
{
    return 2 * tm * 4 * 256 + (nd > 1 ? 3 * 256 : 0) + (epi == kSums ? 0 : tm * (4 / nd) * 512) + PB_MAX_BITS * 4;
}

// Bytes of one staged operand of `rows` digit rows (64 each, and 16 more so that the eight operands that a group of eight
// lanes writes to start in different banks); a tile of a chunk has eight of them
__host__ __device__ inline int stage_operand(int rows) { return rows * 64 + 16; }

// Few digit rows (one or two tiles of sixteen), or small matrices: a wave owns a slice of the columns and turns the words of row
// tile after row tile into codes in its registers; the slices of a row meet in LDS once per row tile.
//   FUSED: the activations are converted in this launch.  Every wave leaves the digits of its slice in LDS, in the order in
//   which the matrix instructions read them, and keeps reading them from there.  Else they come from memory (k_digits).
// Bound: latencies at the small end (launch, activations, weights, barrier), the weight stream at the large end.  The words of
// the next unit are requested before this one is multiplied: 8 KB in flight per wave, sixteen waves.  Turning the words of a unit
// into codes takes 160 operations of the vector ALU, its products 16 (one tile) matrix instructions.
// In a graph, us per call, against the FP4 form that this replaces (two bitlayers and two planes per operand):
// 1024 x 1024, 8 bitlayers, 16 vectors 7.3 -> 4.3; 4096 x 4096, 4 vectors 8.1 -> 6.1; 8192 x 8192, 4 vectors 17.5 -> 14.7; 135 x 69, 7
// bitlayers, 113 vectors 14.7 -> 4.6.  The conversion and the codes of a few vectors are more instructions per wave than their FP4
// operands were, which shows where there is little else: 2 to 4 vectors, one or two bitlayers on wide rows (2002 x 5817, one
// bitlayer, 2 vectors 5.0 -> 5.4), more than eight bitlayers (67 x 6211, 16 bitlayers, 3 vectors of 8 bits 9.5 -> 11.8), and one vector on
// the pairs layout (565 x 14030, two bitlayers 5.6 -> 7.9; 4096 x 4096, 8 bitlayers 5.7 -> 5.1).  2148 drawn calls of several vectors
// are 1.7 times as fast on average, 51 of them slower by more than 1.5 %.

template <int ND, int Q, bool IL, int TM, bool FUSED, int EPI, int POLICY, bool PLAIN>
// (the waves per SIMD: one tile, digits from memory, has four at most where a row has sixteen slices, and the registers that this leaves
// let the compiler request the digits earlier: 67 x 4604, 7 vectors of 16 bits 6.4 -> 5.8 us, 913 x 8013, 15 vectors 7.1 -> 6.7, over 194 drawn
// calls 1.7 % on average)
__global__ __launch_bounds__(stream_waves(TM) * 64)
__attribute__((amdgpu_waves_per_eu(stream_waves(TM) / 4, !FUSED && TM == 1 ? 4 : 8))) void k_i8(const I8Args a)
{
    constexpr int VPT = 16 / ND;            // vectors per tile of sixteen digit rows
    constexpr int VPL = 4 / ND;             // vectors per lane of a result: its four registers are the digits of these
    // four tiles of four digits: tile d is digit d of sixteen vectors.  Else the rows of a tile are, from memory, a digit of four vectors
    // after the other (four lanes next to each other read 64 bytes in one piece: otherwise a load takes several times as long), and
    // as staged a digit of one vector after the other.
    // The digits of one tile are side by side in a register, and the third of four is turned to u ^ 0x80 when they are made: with flags to wait
    // for and a XOR in the loop, as in PLANES, it was slower than with four digits of every value (977 x 10807, 6 bitlayers, 3 vectors
    // 8.4 -> 9.1 us, now 8.1; 870 x 9440, 21 vectors 13.2 -> 13.5, now 12.5).  PLAIN: with them all the same, see launch_imma (pb_act_prep
    // does not know the kernel: two products of 977 x 10807, 3 vectors 14.6 -> 15.5 us).
    constexpr bool PLANES = !FUSED && TM == 4 && ND == 4;
    constexpr bool ONES = ND > 1;
    __shared__ int s_sum[2][TM * 4][64];
    __shared__ int s_ones[3][64];           // sums of the codes, per row
    __shared__ double s_z[TM * VPL][64];
    __shared__ float s_scales[PB_MAX_BITS];
    extern __shared__ __align__(16) unsigned char stage[];
    static_assert(sizeof s_sum + ONES * sizeof s_ones + (EPI != kSums) * sizeof s_z + sizeof s_scales == stream_lds(ND, TM, EPI), "LDS");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = (a.cq + a.chunks_per_wave - 1) / a.chunks_per_wave;   // = blockDim.x / 64
    const int q0 = wave * a.chunks_per_wave;
    const int nq = min(a.chunks_per_wave, a.cq - q0);      // >= 1 by construction
    const int n0 = blockIdx.y * (TM * VPT);
    const int rt0 = blockIdx.x * a.rounds_per_wg;
    const int rounds = min(a.rounds_per_wg, a.rt_count - rt0);   // >= 1 by construction
    const int m = a.m;
    const int kb = lane >> 4, j = lane & 15;

    // ---- the weight stream: units (round, group of bitlayers, chunk) ----
    bool merged = EPI != kSums;             // (until the scales are known)
    struct Unit { int r, f, e, i; };
    auto group_end = [&](int f) {
        const int size = merged ? (f == 0 ? 4 * Q : 4 * Q - 2) : (a.pairs_out ? 2 : 1);
        return min(m, f + size);
    };
    // the next unit; true if it belongs to another group of bitlayers
    auto advance = [&](Unit &u) {
        if (++u.i < nq) return false;
        u.i = 0;
        const int f = u.f;
        u.f = u.e;
        if (u.f == m) { u.f = 0; ++u.r; }
        u.e = group_end(u.f);
        return u.f != f;
    };
    const char *base = reinterpret_cast<const char *>(a.packed) + (size_t)rt0 * a.round_step;
    const uint32_t avail = (uint32_t)(a.packed_bytes - (size_t)rt0 * a.round_step);
    // bitlayer of slot 0 of a group: the group starts at slot 0 (even bitlayer 0) or slot 2
    auto slot0_layer = [](const Unit &u) { return (u.f & ~1) == 0 ? 0 : (u.f & ~1) - 2; };
    // of the group being requested: the records that the descriptor of a slot shows (an absent slot has none: the load returns
    // 0 and moves no data); of the group being multiplied: (IL) which of the two bits of a pair's digits belong to it
    uint32_t records[4 * Q], mask[2 * Q];
    auto request_group = [&](const Unit &u) {
        const int l0 = slot0_layer(u);
#pragma unroll
        for (int s = 0; s < 4 * Q; ++s) {
            const int l = l0 + s, lu = l0 + (s & ~1);
            records[s] = (IL ? lu + 1 >= u.f && lu < u.e : l >= u.f && l < u.e) ? avail : 0u;
        }
    };
    auto multiply_group = [&](const Unit &u) {
        const int l0 = slot0_layer(u);
#pragma unroll
        for (int p = 0; p < 2 * Q; ++p) {
            const int l = l0 + 2 * p;
            mask[p] = (l >= u.f && l < u.e ? 0xAAAAAAAAu : 0u) | (l + 1 >= u.f && l + 1 < u.e ? 0x55555555u : 0u);
        }
    };
    u32x4 ring[2][4 * Q];
    auto issue = [&](u32x4 (&dst)[4 * Q], const Unit &u) {
        const bool ok = u.r < rounds;
        const uint32_t off = (uint32_t)u.r * a.round_step + (uint32_t)(q0 + u.i) * 1024u + (uint32_t)slot0_layer(u) * a.layer_step;
#pragma unroll
        for (int s = 0; s < 4 * Q; ++s) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, ok ? (int)records[s] : 0, 0x00020000);
            dst[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, (int)(off + (uint32_t)s * a.layer_step), POLICY);
        }
    };
    // Layer scales, lane i holds scales[i] and the next one (range-checked: none without scales)
    float scv = 0.0f, scn = 0.0f;
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.scales), 0,
                                                                            a.scales ? m * 4 : 0, 0x00020000);
        scv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, 0, 0));
        scn = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4 + 4, 0, 0));
    }
    uint32_t wide_here = 0;
    if constexpr (PLANES || PLAIN) wide_here = load_wide<TM * VPT / 4>(a, n0 / 4, lane);
    Unit ld = {0, 0, group_end(0), 0};
    request_group(ld);

    for (int i = threadIdx.x; i < 2 * TM * 4 * 64; i += nwaves * 64) (&s_sum[0][0][0])[i] = 0;
    if (ONES)
        for (int i = threadIdx.x; i < 3 * 64; i += nwaves * 64) (&s_ones[0][0])[i] = 0;

    // ---- the digit rows of this wave's chunks ----
    const int operand = stage_operand(a.stage_rows), kbytes = a.stage_rows * 16;
    unsigned char *const my_stage = stage + q0 * TM * 8 * operand;
    if constexpr (FUSED) {
        // two vectors at a time (lane 32 v + 2 word + h, as in k_digits), the next two on their way meanwhile
        const int word = (lane >> 1) & 15, h = lane & 1, vb = lane >> 5;
        const int pairs = min(TM * VPT / 2, (a.act.batch - n0 + 1) / 2), total = pairs * nq;
        const int c0 = 512 * q0 + 32 * word + 4 * h;
        u32x4 v[4], next[4];
        load_columns(a.act, n0 + vb, c0, 512 * (q0 + 1), v);
        __builtin_amdgcn_sched_barrier(0);
        issue(ring[0], ld);
        __builtin_amdgcn_sched_barrier(0);
        int i = 0, p = 0;
#pragma unroll 1
        for (int k = 0; k < total; ++k) {
            int i2 = i, p2 = p + 1;
            if (p2 == pairs) { p2 = 0; ++i2; }
            if (k + 1 < total) load_columns(a.act, n0 + 2 * p2 + vb, c0 + 512 * i2, 512 * (q0 + i2 + 1), next);
            convert_columns(a.act, v);
            u32x4 out[ND];
            byte_digits<ND>(v, out);
            const int tm = p / (VPT / 2), g = p % (VPT / 2);
            unsigned char *dst = my_stage + ((i * TM + tm) * 8 + (word & 3) * 2 + h) * operand + (word >> 2) * kbytes +
                                 (2 * g + vb) * ND * 16;
#pragma unroll
            for (int d = 0; d < ND; ++d) reinterpret_cast<u32x4 *>(dst)[d] = out[d];
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = next[b];
            i = i2; p = p2;
        }
    } else {
        issue(ring[0], ld);
    }
    if (wave == 0 && lane < PB_MAX_BITS) s_scales[lane] = scv;
    if (EPI != kSums) {
        const bool off = lane + 1 < m && !(scv == (lane == 0 ? -2.0f : 2.0f) * scn);
        merged = __builtin_amdgcn_ballot_w64(off) == 0;
        if (!merged) {   // the first unit was requested as a whole group
            ld.e = group_end(0);
            request_group(ld);
            issue(ring[0], ld);
        }
    }
    __syncthreads();   // (the sums are zero)

    // prepared digits: lane 16 kb + row of an operand reads the bytes of digit row % ND of vector row / ND
    // (a top digit that no value needs has no records: the load returns 0 and moves no data)
    const bool wide = !(PLANES || PLAIN) || is_wide(wide_here);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.digits), 0,
                                                                        (int)a.digits_bytes, 0x00020000);
    uint32_t doff[TM], dstep[TM];
    const uint32_t turned = wide && (PLANES || j / 4 == 2) ? 0x80808080u : 0u;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int first = PLANES ? n0 : n0 + tm * VPT, group = first / kGroupVectors, vectors = group_vectors(a.act.batch, group);
        const int v = first % kGroupVectors + (PLANES ? j : j / (4 * ND) * 4 + j % 4), digit = PLANES ? tm : j / 4 % ND;
        doff[tm] = v < vectors && (wide || digit < 3) ? digits_at(group, vectors, a.cq, ND, digit, kb, v) : (uint32_t)kNowhere;
        dstep[tm] = digits_step(vectors, ND);
    }
    // staged digits (rows beyond the staged ones belong to no vector: any digits do)
    const int staged = kb * kbytes + min(j, a.stage_rows - 1) * 16;
    u32x4 areg[2][TM];
    auto load_digits = [&](u32x4 (&dst)[TM], int i, int th) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if constexpr (FUSED)
                dst[tm] = *reinterpret_cast<const u32x4 *>(my_stage + ((i * TM + tm) * 8 + th) * operand + staged);
            else
                dst[tm] = __builtin_amdgcn_raw_buffer_load_b128(rd, (int)doff[tm],
                                                                (int)((uint32_t)((q0 + i) * 8 + th) * dstep[tm]), 0);
        }
    };

    Unit u = ld;
    multiply_group(u);
    int sets = 0;          // (round, group) pairs multiplied so far
    int turn = 0;          // the wave that finishes the first tile of a row tile
    v4i acc[TM], ones;
    float bias_row = 0.0f, c_old = 0.0f;
    // the outputs of a row tile: vectors of a lane, tile after tile; the waves take them in turn
    auto first_item = [&]() { return wave - turn + (wave < turn ? nwaves : 0); };
    auto vector_of = [&](int item) { return PLANES ? n0 + kb * 4 + item : n0 + item / VPL * VPT + kb * VPL + item % VPL; };
    const v4i one = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const Masks masks = make_masks();
    load_digits(areg[0], 0, 0);
    while (u.r < rounds) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (u.r < rounds) {
                if (advance(ld)) request_group(ld);
                // (bias and cell state are requested before the next weights: a wait for them does not wait for those)
                if (a.bias && u.i == nq - 1) bias_row = bias_of(a, (rt0 + u.r) * kTileRows + j);
                if (EPI == kCell && u.i == nq - 1 && u.e == m) {
                    const int row = gates_matrix_row((rt0 + u.r) * kTileRows + j, a.gate_h);
                    c_old = cell_state(a, lane, row, row >= 0, vector_of(first_item()));
                }
                issue(ring[k ^ 1], ld);
                if (u.i == 0) {
                    ones = v4i{0, 0, 0, 0};
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) acc[tm] = v4i{0, 0, 0, 0};
                }
                const uint32_t flip = u.f < 2 ? 0xAAAAAAAAu : 0u;   // (IL) the sign bitlayer is stored complemented
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    uint32_t w[4 * Q];
                    words_of<Q, IL>(ring[k], t, flip, mask, w);
                    v4i b[2];
                    weight_codes<Q, IL, (TM < 4)>(masks, w, b[0], b[1]);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        // the operands of the next step are requested before this step's products
                        if (t < 3 || h == 0) load_digits(areg[h ^ 1], u.i, t * 2 + h + 1);
                        else load_digits(areg[0], ld.i, 0);
                        if constexpr (ONES) ones = __builtin_amdgcn_mfma_i32_16x16x64_i8(one, b[h], ones, 0, 0, 0);
                        if constexpr (PLANES || PLAIN) areg[h][PLANES ? 2 : 0] ^= turned;   // (a branch here costs more: 16 -> 20 us)
#pragma unroll
                        for (int tm = 0; tm < TM; ++tm)
                            acc[tm] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, areg[h][tm]), b[h],
                                                                            acc[tm], 0, 0, 0);
                    }
                }
                if (u.i == nq - 1) {
                    // ---- the group is complete in this wave: the slices of the row meet in LDS ----
                    // Two buffers of sums, used in turn: the wave that finishes a tile clears its sums, and the buffer is
                    // added to again only after the next barrier.  The sums of the codes are read by several waves: three
                    // buffers, each cleared when all have passed the barrier after its reading.
                    const int buf = sets & 1, buf3 = sets % 3;
                    if constexpr (ONES) atomicAdd(&s_ones[buf3][lane], ones[0]);
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                        for (int c = 0; c < 4; ++c) atomicAdd(&s_sum[buf][tm * 4 + c][lane], acc[tm][c]);
                    __syncthreads();
                    ++sets;
                    if (ONES && wave == 0) s_ones[(buf3 + 2) % 3][lane] = 0;
                    const Group g = make_group(a, u.f, u.e, s_scales);
                    const int prow = (rt0 + u.r) * kTileRows + j;
                    const int row = a.gate_h ? gates_matrix_row(prow, a.gate_h) : prow;
                    const bool row_ok = row >= 0 && row < a.R;
                    for (int item = first_item(); item < TM * VPL; item += nwaves) {
                        const int n = vector_of(item), v = kb * VPL + item % VPL;
                        int d[ND];
#pragma unroll
                        for (int c = 0; c < ND; ++c) {
                            int *const at = PLANES ? &s_sum[buf][item + 4 * c][lane]
                                            : FUSED || ND == 1 ? &s_sum[buf][item / VPL * 4 + item % VPL * ND + c][lane]
                                                    : &s_sum[buf][item / VPL * 4 + v % 4][(v / 4 * ND + c) * 16 + j];
                            d[c] = *at;
                            *at = 0;
                        }
                        const int sum1 = ONES ? s_ones[buf3][lane] : 0;
                        if constexpr (EPI == kSums) {
                            store_sum(a, g, row, row_ok, n, integer_sum<ND>(g, d, sum1, wide));
                        } else {
                            double v = scaled_sum<ND>(g, d, sum1, wide);
                            if (!g.first) v += s_z[item][lane];
                            if (!g.last) {
                                s_z[item][lane] = v;
                            } else {
                                if (EPI == kCell && item >= nwaves) c_old = cell_state(a, lane, row, row_ok, n);
                                finish<EPI>(a, lane, row, row_ok, n, v, bias_row, c_old);
                            }
                        }
                    }
                    if (g.last) {
                        turn += TM * VPL;
                        while (turn >= nwaves) turn -= nwaves;
                    }
                }
                if (advance(u)) multiply_group(u);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------

// Digits per value that `act_bits` needs
static int digits_of(int act_bits) { return act_bits <= 8 ? 1 : (act_bits <= 16 ? 2 : 4); }

static ActSource act_source(const float *X0, int cols0, const float *X1, int cols1, int batch, int frac_bits, int act_bits)
{
    ActSource s;
    s.X0 = X0; s.X1 = X1; s.cols0 = cols0; s.cols1 = X1 ? cols1 : 0;
    s.batch = batch;
    s.fscale = ldexpf(1.0f, frac_bits);
    s.imax = (act_bits == 32) ? INT32_MAX : (int32_t)((1u << (act_bits - 1)) - 1u);
    s.imin = -s.imax - 1;
    return s;
}

int launch_digits(const float *X0, int cols0, const float *X1, int cols1, int batch, const Layout &L, int frac_bits,
                  int act_bits, void *digits, void *wide, int32_t *xq_out, bool plain, hipStream_t st)
{
    const ActSource s = act_source(X0, cols0, X1, cols1, batch, frac_bits, act_bits);
    const dim3 grid((unsigned)L.cq, (unsigned)((batch + 3) / 4));
    const uint32_t turn = plain ? 0x80808080u : 0u;
    uint8_t *d = static_cast<uint8_t *>(digits), *w = static_cast<uint8_t *>(wide);
    switch (digits_of(act_bits)) {
        case 1: hipLaunchKernelGGL(k_digits<1>, grid, dim3(128), 0, st, s, L.cq, d, w, xq_out, turn); break;
        case 2: hipLaunchKernelGGL(k_digits<2>, grid, dim3(128), 0, st, s, L.cq, d, w, xq_out, turn); break;
        default: hipLaunchKernelGGL(k_digits<4>, grid, dim3(128), 0, st, s, L.cq, d, w, xq_out, turn); break;
    }
    return (int)hipGetLastError();
}

// [what follows][digits 1, 2, 4][four or eight slots][bits, pairs][way]: digits from memory, one tile or four; converted in the
// launch, one tile or two, one tile with non-temporal loads of the weights; one tile, digits from memory, the third as it stands
// (the sums themselves are asked for in groups of one or two: four slots)
enum { kMemory1 = 0, kMemory4 = 1, kFused1 = 2, kFused2 = 3, kFusedNt = 4, kPlain1 = 5, kStreams = 6 };
static bool is_fused(int way) { return way >= kFused1 && way <= kFusedNt; }
static int way_tiles(int way) { return way == kMemory4 ? 4 : (way == kFused2 ? 2 : 1); }
template <int ND, int Q, bool IL, int TM, bool FUSED, int EPI, int POLICY = 0, bool PLAIN = false>
static const void *stream_kernel()
{
    if constexpr ((EPI == kSums && Q > 1) || (EPI == kCell && IL) || ((POLICY || PLAIN) && EPI != kStore) || (PLAIN && ND != 4)) return nullptr;
    else return reinterpret_cast<const void *>(k_i8<ND, Q, IL, TM, FUSED, EPI, POLICY, PLAIN>);
}
#define PB_I8_IL(ND, Q, IL, E)                                                                                     \
    {stream_kernel<ND, Q, IL, 1, false, E>(), stream_kernel<ND, Q, IL, 4, false, E>(),                              \
     stream_kernel<ND, Q, IL, 1, true, E>(), stream_kernel<ND, Q, IL, 2, true, E>(), stream_kernel<ND, Q, IL, 1, true, E, 2>(), \
     stream_kernel<ND, Q, IL, 1, false, E, 0, true>()}
#define PB_I8_ND(ND, E) {{PB_I8_IL(ND, 1, false, E), PB_I8_IL(ND, 1, true, E)}, {PB_I8_IL(ND, 2, false, E), PB_I8_IL(ND, 2, true, E)}}
#define PB_I8(E) {PB_I8_ND(1, E), PB_I8_ND(2, E), PB_I8_ND(4, E)}
static const void *const kI8[3][3][2][2][kStreams] = {PB_I8(kStore), PB_I8(kCell), PB_I8(kSums)};

// Staged digits of a workgroup at most (a compute unit has 160 KB of LDS)
constexpr int kMaxStage = 140 * 1024;

// Compute units (at least one, or an error); their number does not change while the process lives
static hipError_t compute_units(int *cus)
{
    static int cache;
    *cus = __atomic_load_n(&cache, __ATOMIC_RELAXED);
    if (*cus > 0) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (*cus < 1) return hipErrorInvalidDevice;
    __atomic_store_n(&cache, *cus, __ATOMIC_RELAXED);
    return hipSuccess;
}
// Workgroups of a kernel that a compute unit runs at once (0: the query failed; the answer does not change either).  The query is too high
// twice (256 n workgroups of a kernel that only computes take twice as long from the n on where one more has to wait):
//   It divides the waves of the unit by those of the workgroup.  A workgroup of five to eight waves takes two on every SIMD, one of nine to
//   twelve three: with three places a SIMD one workgroup of five waves runs, not two; with four places two, not three.
//   LDS is given out by 1280 bytes: eleven workgroups of 13120 bytes run, not twelve.
// A grid made for more leaves a rest that runs by itself: 12135 x 2547, 8 bitlayers, 13 vectors (five waves) for two per unit 15.7 us, for one
// 12.5; 10440 x 2457, 6 bitlayers, 55 vectors of 8 bits 16.4, 12.7; 9551 x 2050, 2 bitlayers, 13 vectors of 16 bits for three 9.9, for two 8.8;
// 1731 x 276, 6 bitlayers, 887 vectors of 16 bits (13120 bytes) 19.0, 15.8.
constexpr size_t kLds = 160 * 1024, kLdsPiece = 1280;
static int per_unit(const void *fn, int threads, size_t lds, size_t stage, int *slot)
{
    int v = __atomic_load_n(slot, __ATOMIC_RELAXED);
    if (v > 0) return v;
    if (stage && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxStage) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, fn, threads, stage) != hipSuccess) return 0;
    auto at_most = [&](int n) { v = n < 1 ? 1 : (n < v ? n : v); };
    if (v > 1 && threads > 256) {
        int places = 0;     // waves of a SIMD: workgroups of four waves
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&places, fn, 256, stage) != hipSuccess) return 0;
        at_most(places / ((threads + 255) / 256));
    }
    if (v > 1) at_most((int)(kLds / ((lds + stage + kLdsPiece - 1) / kLdsPiece * kLdsPiece)));
    if (v > 0) __atomic_store_n(slot, v, __ATOMIC_RELAXED);
    return v;
}

// The call as the choice of the kernel sees it
struct I8Call {
    int rt, cq, tiles, batch, nd, m, groups;
    double weights;   // MB of packed words
};
static int stage_rows(const I8Call &c, int tm)
{
    const int rows = c.nd * ((c.batch + 1) & ~1);   // (vectors are converted two at a time)
    return tm > 1 || rows > 16 ? 16 : rows;
}
static size_t stage_bytes(const I8Call &c, int tm) { return (size_t)c.cq * (size_t)(tm * 8 * stage_operand(stage_rows(c, tm))); }
static int slice(int cq, int tm) { return (cq + stream_waves(tm) - 1) / stream_waves(tm); }   // chunks per wave

// Workgroups of S waves per compute unit of the kernels that convert the activations: each repeats the conversion, so no more than
// eight waves need.  (5003 x 3001, 5 vectors of 16 bits, six waves: one per compute unit 7.5 us, two 8.6; 4096 x 1024, 16
// vectors, two waves: one 7.5, two 6.8, four 5.8 us.)
static int fused_per_cu(int S) { return S >= 4 ? 1 : 8 / S; }

// Weights that are read once (one tile of digit rows): non-temporal loads, which find them in the last-level cache but leave nothing
// there.  Graph of calls, 8 bitlayers, 8192 columns, two vectors, plain / non-temporal loads in us where something else has put the
// weights there (packing) / where only the calls themselves read them, after 1 GB of other data:
//   33 MB 7.9 / 8.0, 8.0 / 10.0    40 MB 11.0 / 11.3, 11.3 / 12.8    48 MB 12.6 / 11.8, 12.8 / 13.1    56 MB 13.4 / 12.9, 13.5 / 14.6
//   64 MB 14.4 / 13.1, 14.6 / 14.4    76 MB 16.6 / 16.3, 16.6 / 17.2    90 MB 18.2 / 18.6, 18.2 / 19.7
// (3072 columns, 5 vectors of 16 bits: 34 MB 9.4 / 9.5, 9.4 / 10.4; 48 MB 12.4 / 11.5, 12.5 / 12.1; 64 MB 15.0 / 14.8, 15.2 / 15.4)
static bool streaming(const I8Call &c) { return c.tiles == 1 && c.weights > 44.0 && c.weights <= 72.0; }

// Which kernel: the one with the least estimated time.  The estimates are in us, fitted to the times of 280 layers on an MI355X (64
// to 16384 rows, 64 to 32768 columns, 2 to 1024 vectors, 1 to 16 bitlayers, 8, 16 and 32 activation bits, both layouts).  Over 2148 other
// calls with every kernel timed, the choice costs 2.6 % on average over the best one, 19 % at the 95th percentile, 1.85 times in
// the worst case: it is weakest with 8- and 16-bit activations of many vectors on a small matrix, whose conversion one after the other
// the estimate takes for shorter than it is (284 x 1200, 21 vectors of 8 bits, cell update 12.2 us, from memory 6.9).  A term for that
// chain, fitted to 900 of the calls, moved 62 of the other 1500 to a kernel over 3 % slower and 48 to one as much faster: left out.
// With digits by groups of sixteen vectors and three of four, 420 more calls: 3.3 % on average over the best, 19 %, 1.55 times; fitted again to
// half of them the estimates were no better on the other half (3.1 %, 3.0 % before) and stay.
// The bitlayers count by themselves: with one cost for all,
// one and two bitlayers of a few vectors went to the wrong kernel (3841 x 7174, one bitlayer, 14 vectors: 13.4 us, here 10.9).
//   few digit rows: rounds of workgroups over the chip (16 / S at once, which they were fitted with; per_unit has what runs), units
//                   (row tile, group, tile of digit rows, chunk), conversion
//   many:           rounds of workgroups times (start and end + steps), the digits of all vectors through memory
static int pick_way(const I8Call &c, bool prepared, int cus)
{
#ifdef PB_TUNING
    if (const char *e = getenv("PB_TUNE_WAY")) {
        const int w = atoi(e);
        if (w >= 0 && (!is_fused(w) || (!prepared && stage_bytes(c, way_tiles(w)) <= kMaxStage))) return w;
    }
#endif
    int best = kMemory1;
    double least = 1e30;
    auto offer = [&](int way, double t) {
        if (t < least) { least = t; best = way; }
    };
    const double bits = (c.m < 8 ? c.m : 8) / 8.0;
    const double quad = c.m > 4 ? 4.0 : 2.0;       // (the codes of a unit cost about as much as that many matrix tiles)
    for (int way = 0; way < kFusedNt; ++way) {
        const int tm = way_tiles(way), groups = (c.tiles + tm - 1) / tm;
        const size_t lds = is_fused(way) ? stage_bytes(c, tm) : 0;
        if (is_fused(way) && (prepared || lds > kMaxStage)) continue;
        const int cpw = slice(c.cq, tm), S = (c.cq + cpw - 1) / cpw;
        int per_cu = is_fused(way) ? fused_per_cu(S) : 16 / S;
        if (is_fused(way) && (size_t)per_cu * (lds + 4096) > 155 * 1024) per_cu = (int)(155 * 1024 / (lds + 4096));
        const int cap = cus * (per_cu < 1 ? 1 : per_cu);
        int wgs = cap / groups < 1 ? 1 : cap / groups;
        if (wgs > c.rt) wgs = c.rt;
        const int rounds = (c.rt + wgs - 1) / wgs;
        const int waves = (((c.rt + rounds - 1) / rounds) * groups + cap - 1) / cap;   // (workgroups after another on a place)
        const double sets = (double)waves * rounds * c.groups;
        const double units = (double)c.rt * groups * c.cq * c.groups * (1.0 + tm / quad) / 1000.0;
        const int pairs = (c.batch + 1) / 2 < 8 * tm / c.nd ? (c.batch + 1) / 2 : 8 * tm / c.nd;     // of vectors of a workgroup
        const double conversions = (double)((((c.rt + rounds - 1) / rounds) * groups + cus - 1) / cus) * c.cq * pairs / 10.0;
        const double digits = c.tiles * c.cq / 100.0;
        const double steps = sets * cpw;
        switch (way) {
        case kMemory1: offer(way, (prepared ? 2.9 : 4.9) + 1.34 * steps + 1.51 * digits + (0.10 + 0.27 * bits) * units + 0.051 * c.weights); break;
        case kMemory4: offer(way, (prepared ? 3.6 : 5.6) + (1.55 + 0.48 * bits) * steps + 1.33 * digits + (0.24 + 0.34 * bits) * units + 0.019 * c.weights); break;
        case kFused1: offer(way, 3.4 + (0.60 + 0.37 * bits) * steps + 0.69 * conversions + (0.20 + 0.15 * bits) * units); break;
        default: offer(way, 3.4 + 0.69 * bits * steps + 0.87 * sets + 0.79 * conversions + 0.137 * units); break;
        }
    }
    static const double cost[kTileShapes][5] = {   // start, step, start and end of a workgroup, weights (MB), digits
        {3.4, 1.67, 5.79, 0.074, 0.0094}, {3.6, 2.68, 7.80, 0.060, 0.0075}, {2.9, 4.31, 17.0, 0.100, 0.0143}};
    for (int i = 0; i < kTileShapes; ++i) {
        const TileShape &t = kTile[i];
        if (c.groups > t.nt) continue;      // (a row tile's groups would take several passes)
        const int rows = t.nt / c.groups;
        const int wgs = ((c.rt + rows - 1) / rows) * ((c.tiles + t.nt * t.tm - 1) / (t.nt * t.tm));
        const int rounds = (wgs + cus - 1) / cus;
        const int per_step = 8 / t.nt;      // chunks
        const int steps = (c.cq + per_step - 1) / per_step;
        offer(kStreams + i, cost[i][0] + rounds * (cost[i][2] + steps * cost[i][1]) + cost[i][3] * c.weights + cost[i][4] * c.tiles * c.cq);
    }
    return best == kFused1 && streaming(c) ? kFusedNt : best;
}

int launch_imma(const uint32_t *packed, const float *scales, const Layout &L, int bits_used, int frac_bits, int act_bits,
                const float *X0, int cols0, const float *X1, int cols1, void *digits, void *wide, bool prepared, int batch,
                float *Y, long long *A, bool pairs_out, const Epilogue &ep, hipStream_t st)
{
    const int nd = digits_of(act_bits);
    I8Args a;
    a.packed = packed;
    a.packed_bytes = (uint32_t)packed_bytes(L);   // (the host API refuses matrices of 4 GiB and more)
    a.layer_step = (uint32_t)(tile16_layer_stride(L) * 4);
    a.round_step = (uint32_t)(tile16_rowtile_stride(L) * 4);
    a.rt_count = L.rt_count; a.cq = L.cq; a.m = bits_used;
    a.digits = static_cast<const uint8_t *>(digits);
    a.digits_bytes = (uint32_t)batch * (uint32_t)L.cq * (uint32_t)(nd * 512);
    a.wide = static_cast<const uint8_t *>(wide);
    a.act = act_source(X0, cols0, X1, cols1, batch, frac_bits, act_bits);
    a.scales = scales; a.Y = Y; a.A = A; a.pairs_out = (A && pairs_out) ? 1 : 0;
    a.bias = ep.bias; a.relu = ep.relu; a.c_prev = ep.c_prev; a.h_out = ep.h_out; a.c_out = ep.c_out;
    a.gate_h = L.gate_h; a.R = L.rows;
    a.out_scale = ldexp(1.0, -frac_bits);
    // (the epilogue addresses the bias and the cell state with 32-bit byte offsets)
    if (ep.bias && L.rows >= (1 << 29)) return (int)hipErrorInvalidValue;
    if (ep.c_prev && (size_t)batch * (size_t)L.gate_h >= ((size_t)1 << 29)) return (int)hipErrorInvalidValue;

    const int vpt = 16 / nd;
    const bool il = is_pairs(L.layout);
    I8Call c;
    c.rt = L.rt_count; c.cq = L.cq; c.tiles = (batch + vpt - 1) / vpt; c.batch = batch; c.nd = nd; c.m = bits_used;
    c.groups = A ? (pairs_out ? (bits_used + 1) / 2 : bits_used) : i8_groups(bits_used);
    c.weights = (double)L.layer_words * 4e-6 * bits_used;
    int cus;
    const hipError_t no_device = compute_units(&cus);
    if (no_device != hipSuccess) return (int)no_device;
    int way = pick_way(c, prepared, cus);
    if (way == kFusedNt && (A || ep.c_prev)) way = kFused1;
    // Third digits as they stand: what pb_act_prep leaves; and with at most four bitlayers and more than four tiles, whose digits take longer to read
    // than flags and XOR (1291 x 9493, 4 bitlayers, 17 vectors 11.5 us, all four digits 12.4; 393 x 14185, 2 bitlayers, 29 vectors 9.5, 9.9;
    // but 16337 x 1799, 4 bitlayers, 3 vectors 6.9, 6.5, and 870 x 9440, 8 bitlayers, 21 vectors 13.5, 12.5).
    if (way == kMemory1 && nd == 4 && (prepared || (c.tiles > 4 && bits_used <= 4 && !A && !ep.c_prev))) way = kPlain1;
    const int shape = way - kStreams;
    if (!prepared && !is_fused(way)) {
        const int e = launch_digits(X0, cols0, X1, cols1, batch, L, frac_bits, act_bits, digits, wide, nullptr, way != kMemory1, st);
        if (e) return e;
    }
    if (shape >= 0) return launch_imma_tile(shape, a, nd, il, st);

    const int epi = A ? kSums : (ep.c_prev ? kCell : kStore), q = (!A && bits_used > 4) ? 1 : 0;
    const int ndi = nd == 4 ? 2 : nd - 1, tm = way_tiles(way);
    const void *fn = kI8[epi][ndi][q][il][way];
    if (!fn) return (int)hipErrorInvalidValue;
    a.chunks_per_wave = slice(L.cq, tm);
    a.stage_rows = stage_rows(c, tm);
    const int S = (L.cq + a.chunks_per_wave - 1) / a.chunks_per_wave;
    const size_t lds = is_fused(way) ? stage_bytes(c, tm) : 0;
    static int cache[3][3][2][2][kStreams][17][24];   // (the last index: LDS in steps of 6 KB)
    int most = per_unit(fn, S * 64, (size_t)stream_lds(nd, tm, epi), lds, &cache[epi][ndi][q][il][way][S][lds / 6144]);
    if (most < 1) return (int)hipErrorInvalidValue;
    if (is_fused(way) && most > fused_per_cu(S)) most = fused_per_cu(S);
    const int groups = (c.tiles + tm - 1) / tm;
    // Workgroups, and the row tiles of each: as many as run at once.  Of those with more than four waves fewer where the unit that does the most
    // then has fewer row tiles to do: 9619 x 11869, one bitlayer, 16 vectors (eight waves, pairs layout) two workgroups of two row tiles 33.6 us, one
    // of three 30.1; 5888 x 3649, 3 bitlayers, 11 vectors of 16 bits 9.0, 8.5.  With as many to do, two at once are faster than one:
    // 14587 x 2129, 3 bitlayers, 51 vectors of 8 bits (five waves) two of two 12.4, one of four 15.5.
    int wgs = 1;
    for (int n = most, least = INT32_MAX; n >= 1; --n) {
        int w = cus * n / groups;
        w = w < 1 ? 1 : (w < L.rt_count ? w : L.rt_count);
        const int rounds = (L.rt_count + w - 1) / w;
        w = (L.rt_count + rounds - 1) / rounds;
        const int cost = rounds * (6 + (w * groups + cus - 1) / cus * S);
        if (cost < least) { least = cost; wgs = w; a.rounds_per_wg = rounds; }
        if (S <= 4 || is_fused(way)) break;
    }
    void *args[] = {&a};
    const hipError_t e = hipLaunchKernel(fn, dim3((unsigned)wgs, (unsigned)groups), dim3((unsigned)S * 64), args, lds, st);
    return (int)(e != hipSuccess ? e : hipGetLastError());
}

}  // namespace pb
