// The product on the 8-bit integer matrix cores for many digit rows (see pb_imma.h for the arithmetic).
#include <type_traits>

#include "pb_imma.h"

namespace pb {

// Many digit rows: the eight waves of a workgroup share the expanded weight codes through LDS.
//   NT waves lie along the digit rows, TM tiles of sixteen each; 8 / NT groups of waves share out the columns.  A tile is one digit
//   of sixteen vectors: a wave of four tiles has all digits of sixteen vectors of 32 bits, and of two waves of two tiles one has the
//   lower two and the other the upper two.  Sixteen vectors that need only three digits cost three tiles: the fourth is neither read
//   nor multiplied, and the waves are numbered so that every SIMD has as many waves of lower as of upper digits.
//   NT column slots (a row tile and a group of bitlayers each); a step of a group of waves covers a chunk of 512 columns,
//   and every wave expands one unit (slot, chunk) per step: it loads the words two steps ahead, turns them into codes
//   one step ahead, and multiplies its own digit rows, which come straight from memory (each byte is used by one
//   wave only), with the codes of all units of the step.
// Bound: the matrix instructions at the large end (one in 16 cycles per SIMD); for few vectors the digit rows, which every
// workgroup reads at 64 bytes per cycle, LDS, the expansion and the matrix instructions, about as long each.  Operands of the codes
// are read from LDS three (six, seven) products ahead and the scheduler is kept from moving work across a (t, h): without that barrier
// the products waited for their operands (64 vectors: 39 -> 32 us).
// us per call in a graph, digits included, 8192 x 8192, 8 bitlayers, values within three digits, against four digits with a vector's digits
// next to each other in memory: 16 vectors 24.4 -> 22.3, 64 31.2 -> 28.1, 256 74.9 -> 64.6, 1024 260 -> 214 (pairs layout 261 -> 214);
// 16384 x 16384, 64 vectors 117 -> 103, 256 255 -> 214.  Vectors of 8 bits, whose rows now are four pieces of 256 bytes and were sixteen
// of 64: 64 vectors 41.5 -> 23.4, 256 47.2 -> 34.6, 1024 94.6 -> 85.1; of 16 bits 30.8 -> 28.0, 63.7 -> 60.5, 151 -> 149.
// Values beyond three digits, one in every sixteen vectors, against four digits of every value as it was: 64 vectors 31.3 -> 30.2, 256 73.9 -> 71.5,
// 1024 260 -> 248; 3795 x 5918, 16 bitlayers, 301 vectors 133.8 -> 133.6.
// A kernel for each number of digits: one kernel for all of them had the loop over the steps three times and every kind of output, which
// filled the registers (scratch memory also in the shape of eight waves and two tiles), and turned a digit of 8- and 16-bit vectors by zero.
// One kernel -> three: 64 vectors 28.0 -> 27.3, with values beyond three digits 30.8 -> 30.2, 4096 x 4096 16.5 -> 15.8; 1024 vectors of 8 bits 86.4 ->
// 84.0, 256 34.7 -> 34.0; LSTM step 6000 x 3000, 5 bitlayers, 64 vectors 18.3 -> 17.3.
// The shape with four tiles per wave still needs more than the 256 registers of a wave (up to 196 bytes of scratch): the loop of three digits
// has none of them, those of four, two and one reload up to twelve registers in a step of 264 matrix instructions.  A kernel with scratch takes
// 0.3 us longer to launch.
// Calls with several groups of bitlayers (more than eight bitlayers, scales that do not halve, the parity hooks) give them
// slots of their own, so that the sums of a row tile's groups meet in a lane.
template <int ND, int Q, bool IL, int NT, int TM, int EPI>
__global__ __launch_bounds__(512) void k_i8_tile(const I8Args a, const int rows_per_wg)
{
    constexpr int nds = ND == 4 ? 2 : ND - 1;
    constexpr int WK = 8 / NT;
    constexpr int UNIT = 8 * 1024;          // codes of a unit: eight operands of 1 KB
    constexpr int BUF = 8 * UNIT;
    constexpr int BR = TM >= 4 ? 4 : (NT == 8 ? 7 : 8);     // operands of codes: ring
    constexpr int AR = NT * TM >= 32 ? 2 : 4;     // operands of digit rows: ring of steps (t, h)
    extern __shared__ __align__(16) unsigned char lds[];    // two buffers
    __shared__ int s_ones[NT][64];
    __shared__ float s_bias[NT][kTileRows];
    __shared__ float s_scales[PB_MAX_BITS];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % NT, kg = wave / NT;     // (the wave's digit rows and the slot that it expands; its columns)
    const int kb = lane >> 4, j = lane & 15;
    const int m = a.m;
    // its tiles: digit and group of vectors of each
    const int role = WK == 2 && kg == 1 ? NT - 1 - wm : wm;
    constexpr bool halves = TM == 2 && ND == 4;      // (two waves share a group's digits)
    const int half = halves ? role / (NT / 2) : 0;
    int group[TM], digit[TM];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int tile = ((int)blockIdx.y * NT + role) * TM + tm;
        group[tm] = halves ? (int)blockIdx.y * (NT / 2) + role % (NT / 2) : tile >> nds;
        digit[tm] = halves ? 2 * half + tm : tile & ((1 << nds) - 1);
    }
    const int rt0 = blockIdx.x * rows_per_wg;
    const int rts = min(rows_per_wg, a.rt_count - rt0);     // >= 1 by construction
    const int steps = (a.cq + WK - 1) / WK;
    const Masks masks = make_masks();

    float scv, scn;
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.scales), 0,
                                                                            a.scales ? m * 4 : 0, 0x00020000);
        scv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, 0, 0));
        scn = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4 + 4, 0, 0));
    }
    const uint32_t wide_here = nds == 2 ? load_wide<4>(a, group[0] * 4, lane) : 0;
    if (wave == 0 && lane < PB_MAX_BITS) s_scales[lane] = scv;
    bool merged = false;
    if (EPI != kSums) {
        const bool off = lane + 1 < m && !(scv == (lane == 0 ? -2.0f : 2.0f) * scn);
        merged = __builtin_amdgcn_ballot_w64(off) == 0;
    }
    const int gs0 = merged ? 4 * Q : (EPI == kSums && a.pairs_out ? 2 : 1), gs1 = merged ? 4 * Q - 2 : gs0;
    int ng = 1;                                 // groups of a row tile
    for (int f = gs0; f < m; f += gs1) ++ng;
    auto group_first = [&](int g) { return g == 0 ? 0 : gs0 + (g - 1) * gs1; };
    auto group_end = [&](int g) { return min(m, gs0 + g * gs1); };
    int rp = 1;                                 // row tiles of a pass
    while ((rp + 1) * ng <= NT) ++rp;
    const bool carry = ng > NT;                 // (a row tile's groups take several passes, its sums wait in the second buffer)

    // digit rows
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(a.digits), 0,
                                                                        (int)a.digits_bytes, 0x00020000);
    uint32_t doff[TM], dstep[TM];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int vectors = group_vectors(a.act.batch, group[tm]);
        doff[tm] = j < vectors ? digits_at(group[tm], vectors, a.cq, 1 << nds, digit[tm], kb, j) : (uint32_t)kNowhere;
        dstep[tm] = digits_step(vectors, 1 << nds);
    }
    // whether the top digits count (where a row tile's groups take several passes they always do), and then the digits to be turned
    const bool wide = nds == 2 && (carry || is_wide(wide_here));
    const bool turns = wide && (TM == 4 || half == 1);
    const char *base = reinterpret_cast<const char *>(a.packed) + (size_t)rt0 * a.round_step;
    const uint32_t avail = (uint32_t)(a.packed_bytes - (size_t)rt0 * a.round_step);

    for (int r = 0, g0 = 0; r < rts;) {
        const int slots = carry ? min(NT, ng - g0) : min(rp, rts - r) * ng;
        // this wave's unit: row tile my_r, group my_g
        int my_r = r, my_g = g0 + wm;
        if (!carry)
            while (my_g >= ng) { my_g -= ng; ++my_r; }
        const bool have = wm < slots;
        const int f = group_first(my_g), e = group_end(my_g);
        const int l0 = (f & ~1) == 0 ? 0 : (f & ~1) - 2;
        uint32_t mask[2 * Q];
#pragma unroll
        for (int p = 0; p < 2 * Q; ++p) {
            const int l = l0 + 2 * p;
            mask[p] = !have ? 0u
                            : (l >= f && l < e ? 0xAAAAAAAAu : 0u) | (l + 1 >= f && l + 1 < e ? 0x55555555u : 0u);
        }
        const uint32_t flip = l0 == 0 ? 0xAAAAAAAAu : 0u;
        u32x4 w[4 * Q];
        auto issue = [&](int step) {
            const int q = step * WK + kg;
            const uint32_t off = (uint32_t)my_r * a.round_step + (uint32_t)q * 1024u;
#pragma unroll
            for (int s = 0; s < 4 * Q; ++s) {
                const int l = l0 + s, lu = l0 + (s & ~1);
                const bool has = IL ? lu + 1 >= f && lu < e : l >= f && l < e;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<char *>(base), 0, have && has && q < a.cq ? (int)avail : 0, 0x00020000);
                w[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, (int)(off + (uint32_t)l * a.layer_step), 0);
            }
        };
        v4i ones = v4i{0, 0, 0, 0};
        const v4i one = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
        unsigned char *const my_codes = lds + wave * UNIT + lane * 16;
        // word t of the unit of `step` -> codes
        auto expand = [&](int t, int step, int buf) {
            const bool in = step * WK + kg < a.cq;
            uint32_t keep[2 * Q], p[4 * Q];
#pragma unroll
            for (int i = 0; i < 2 * Q; ++i) keep[i] = in ? mask[i] : 0u;
            words_of<Q, IL>(w, t, flip, keep, p);
            v4i lo, hi;
            weight_codes<Q, IL, true>(masks, p, lo, hi);
            ones = __builtin_amdgcn_mfma_i32_16x16x64_i8(one, lo, ones, 0, 0, 0);
            ones = __builtin_amdgcn_mfma_i32_16x16x64_i8(one, hi, ones, 0, 0, 0);
            *reinterpret_cast<v4i *>(my_codes + buf * BUF + t * 2048) = lo;
            *reinterpret_cast<v4i *>(my_codes + buf * BUF + t * 2048 + 1024) = hi;
        };
        u32x4 ar[AR][TM];
        auto load_digits = [&](auto tiles, u32x4 (&dst)[TM], int step, int th) {
            // (beyond the last chunk the codes are zero: any digits do)
            const int q = min(step * WK + kg, a.cq - 1);
#pragma unroll
            for (int tm = 0; tm < decltype(tiles)::value; ++tm)
                dst[tm] = __builtin_amdgcn_raw_buffer_load_b128(rd, (int)doff[tm], (int)((uint32_t)(q * 8 + th) * dstep[tm]), 0);
        };
        v4i acc[TM][NT];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[tm][nt] = v4i{0, 0, 0, 0};
        // the codes of slot nt, operand th
        auto codes = [&](int buf, int th, int nt) {
            return *reinterpret_cast<const v4i *>(lds + buf * BUF + (kg * NT + nt) * UNIT + th * 1024 + lane * 16);
        };
        auto multiply = [&](auto tiles, const u32x4 (&dig)[TM], const v4i b, int nt) {
#pragma unroll
            for (int tm = 0; tm < decltype(tiles)::value; ++tm)
                acc[tm][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, dig[tm]), b, acc[tm][nt], 0, 0, 0);
        };
        for (int i = threadIdx.x; i < NT * 64; i += 512) (&s_ones[0][0])[i] = 0;
        if (threadIdx.x < NT * kTileRows) {
            int nt = threadIdx.x / kTileRows, rr = r;
            if (!carry)
                while (nt >= ng) { nt -= ng; ++rr; }
            s_bias[threadIdx.x / kTileRows][j] = EPI != kSums && a.bias ? bias_of(a, (rt0 + rr) * kTileRows + j) : 0.0f;
        }
        issue(0);
        constexpr int XT = TM == 4 ? 2 : 0;         // the tile of digit 2 (if it is of four)
        // the steps with the first `tiles` tiles of the wave; `turn`: digit 2 has to be turned
        auto products = [&](auto tiles, auto turn) {
#pragma unroll
            for (int k = 0; k < AR - 1; ++k) load_digits(tiles, ar[k], 0, k);
#pragma unroll
            for (int t = 0; t < 4; ++t) expand(t, 0, 0);
            issue(1);
            __syncthreads();
            for (int step = 0; step < steps; ++step) {
                const int buf = step & 1;
                // (the codes of BR - 1 operands ahead are on their way from LDS)
                v4i br[BR];
#pragma unroll
                for (int i = 0; i < BR - 1; ++i) br[i] = codes(buf, i / NT, i % NT);
#pragma unroll
                for (int th = 0; th < 8; ++th) {
                    // the digit rows of a later (t, h) are requested before this one's products
                    const int nx = th + AR - 1;
                    if (nx < 8) load_digits(tiles, ar[nx % AR], step, nx);
                    else load_digits(tiles, ar[nx % AR], step + 1, nx - 8);
                    if ((th & 1) == 0) expand(th / 2, step + 1, buf ^ 1);
                    if (th == 7) issue(step + 2);
                    if constexpr (decltype(turn)::value) ar[th % AR][XT] ^= 0x80808080u;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const int i = th * NT + nt, ahead = i + BR - 1;
                        if (ahead < 8 * NT) br[ahead % BR] = codes(buf, ahead / NT, ahead % NT);
                        multiply(tiles, ar[th % AR], br[i % BR], nt);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
            }
        };
        const std::integral_constant<int, TM> all;
        const std::integral_constant<int, TM - 1> but_one;
        if (!carry) {
            if constexpr (ND != 4) products(all, std::false_type{});
            else if (!wide && (TM == 4 || half == 1)) products(but_one, std::false_type{});
            else if (turns) products(all, std::true_type{});
            else products(all, std::false_type{});
        } else {
            for (int step = 0; step < steps; ++step) {
#pragma unroll
                for (int t = 0; t < 4; ++t) expand(t, step, 0);
                issue(step + 1);
                __syncthreads();
                for (int th = 0; th < 8; ++th) {
                    load_digits(all, ar[0], step, th);
                    if constexpr (ND == 4) ar[0][XT] ^= turns ? 0x80808080u : 0u;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) multiply(all, ar[0], codes(0, th, nt), nt);
                }
                __syncthreads();
            }
        }
        // ---- the groups of waves add up, then every tile is finished ----
        atomicAdd(&s_ones[wm][lane], ones[0]);
        int *const part = reinterpret_cast<int *>(lds) + role * (TM * NT * 4 * 64) + lane;
        for (int k = 1; k < WK; ++k) {
            if (k > 1) __syncthreads();
            if (kg == k) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                        for (int c = 0; c < 4; ++c) part[((nt * TM + tm) * 4 + c) * 64] = acc[tm][nt][c];
            }
            __syncthreads();
            if (kg == 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[tm][nt][c] += part[((nt * TM + tm) * 4 + c) * 64];
            }
        }
        __syncthreads();
        // Two waves of a group's digits: each finishes every other row tile, and leaves its sums of the others in LDS.
        int *const shared = reinterpret_cast<int *>(lds) + role % (NT / 2) * (TM * NT * 4 * 64) + lane;
        auto mine = [&](int rr) { return !halves || ((rr - r) & 1) == half; };
        if (halves) {
            if (kg == 0) {
                int rr = r, gg = g0;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if (!mine(rr)) {
#pragma unroll
                        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                            for (int c = 0; c < 4; ++c) shared[((nt * TM + tm) * 4 + c) * 64] = acc[tm][nt][c];
                    }
                    if (++gg == ng) { gg = 0; ++rr; }
                }
            }
            __syncthreads();
        }
        if (kg == 0) {
            int rr = r, gg = g0;
            for (int nt = 0; nt < slots; ++nt) {
                if (mine(rr)) {
                    const Group g = make_group(a, group_first(gg), group_end(gg), s_scales);
                    const int sum1 = s_ones[nt][lane];
                    const float bias_row = s_bias[nt][j];
                    int d[TM][4] = {};
#pragma unroll
                    for (int x = 0; x < NT; ++x)
                        if (x == nt) {
#pragma unroll
                            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                                for (int c = 0; c < 4; ++c) d[tm][c] = acc[tm][x][c];
                        }
                    const int prow = (rt0 + rr) * kTileRows + j;
                    const int row = a.gate_h ? gates_matrix_row(prow, a.gate_h) : prow;
                    const bool row_ok = row >= 0 && row < a.R;
                    // `digits` tiles of this wave have the digits of four vectors of the lane, the lowest first
                    auto outputs = [&](auto digits, auto both) {
                        constexpr int OWN = decltype(both)::value ? 2 : ND, VECTORS = TM / OWN * 4;
                        auto vector = [&](int i) { return group[i / 4 * OWN] * kGroupVectors + kb * 4 + i % 4; };
                        float c_old[VECTORS] = {};
                        if (EPI == kCell && g.last) {
#pragma unroll
                            for (int i = 0; i < VECTORS; ++i) c_old[i] = cell_state(a, lane, row, row_ok, vector(i));
                        }
#pragma unroll
                        for (int i = 0; i < VECTORS; ++i) {
                            int dd[ND];
#pragma unroll
                            for (int k = 0; k < OWN; ++k) dd[k] = d[i / 4 * OWN + k][i % 4];
                            if constexpr (decltype(both)::value) {
#pragma unroll
                                for (int k = 0; k < 2; ++k) {
                                    const int own = dd[k], other = shared[((nt * TM + k) * 4 + i) * 64];
                                    dd[k] = half ? other : own;
                                    dd[2 + k] = half ? own : other;
                                }
                            }
                            if constexpr (EPI == kSums) {
                                store_sum(a, g, row, row_ok, vector(i), integer_sum<ND>(g, dd, sum1, wide));
                            } else {
                                double *z = reinterpret_cast<double *>(lds + BUF) + (wm * TM * 4 + i) * 64 + lane;
                                double v = scaled_sum<ND>(g, dd, sum1, wide);
                                if (!g.first) v += *z;
                                if (!g.last) *z = v;
                                else finish<EPI>(a, lane, row, row_ok, vector(i), v, bias_row, c_old[i]);
                            }
                        }
                    };
                    outputs(std::integral_constant<int, ND>{}, std::integral_constant<bool, halves>{});
                }
                if (++gg == ng) { gg = 0; ++rr; }
            }
        }
        __syncthreads();
        if (!carry) r += rp;
        else if ((g0 += NT) >= ng) { g0 = 0; ++r; }
    }
}


// ---------------------------------------------------------------------------------------------------------------

template <int ND, int Q, bool IL, int NT, int TM, int EPI>
static const void *tile_kernel()
{
    // (the sums themselves are asked for in groups of one or two: four slots)
    if constexpr ((EPI == kSums && Q > 1) || (EPI == kCell && IL)) return nullptr;
    else return reinterpret_cast<const void *>(k_i8_tile<ND, Q, IL, NT, TM, EPI>);
}
#define PB_TILE_E(ND, NT, TM, E) {{tile_kernel<ND, 1, false, NT, TM, E>(), tile_kernel<ND, 1, true, NT, TM, E>()}, \
                                  {tile_kernel<ND, 2, false, NT, TM, E>(), tile_kernel<ND, 2, true, NT, TM, E>()}}
#define PB_TILE_ND(ND, NT, TM) {PB_TILE_E(ND, NT, TM, kStore), PB_TILE_E(ND, NT, TM, kCell), PB_TILE_E(ND, NT, TM, kSums)}
#define PB_TILE(NT, TM) {PB_TILE_ND(1, NT, TM), PB_TILE_ND(2, NT, TM), PB_TILE_ND(4, NT, TM)}
static const void *const kTileFn[kTileShapes][3][3][2][2] = {PB_TILE(4, 2), PB_TILE(8, 2), PB_TILE(8, 4)};
constexpr int kTileLds = 128 * 1024;

int launch_imma_tile(int shape, const I8Args &a, int nd, bool il, hipStream_t st)
{
    const int epi = a.A ? kSums : (a.c_prev ? kCell : kStore), q = (epi != kSums && a.m > 4) ? 1 : 0, ndi = nd == 4 ? 2 : nd - 1;
    const void *fn = kTileFn[shape][ndi][epi][q][il];
    static bool declared[kTileShapes][3][3][2][2];
    if (!fn) return (int)hipErrorInvalidValue;
    if (!__atomic_load_n(&declared[shape][ndi][epi][q][il], __ATOMIC_RELAXED)) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds);
        if (e != hipSuccess) return (int)e;
        __atomic_store_n(&declared[shape][ndi][epi][q][il], true, __ATOMIC_RELAXED);
    }
    const TileShape &t = kTile[shape];
    int rows_per_wg = tile_rows(t, a.m, epi == kSums);
    const int vpt = 16 / nd, tiles = (a.act.batch + vpt - 1) / vpt;
    const int groups = (tiles + t.nt * t.tm - 1) / (t.nt * t.tm), wgs = (a.rt_count + rows_per_wg - 1) / rows_per_wg;
    void *args[] = {const_cast<I8Args *>(&a), &rows_per_wg};
    const hipError_t e = hipLaunchKernel(fn, dim3((unsigned)wgs, (unsigned)groups), dim3(512), args, kTileLds, st);
    return (int)(e != hipSuccess ? e : hipGetLastError());
}

}  // namespace pb
