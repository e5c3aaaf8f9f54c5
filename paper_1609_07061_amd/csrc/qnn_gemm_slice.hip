// Matrix-core kernel for products that do not fill the chip with large tiles, or whose rows are not made of whole aligned
// groups: small batches, single time steps, odd layer widths, convolutions of a few images.
//
// Bound: latency.  Such a product is a few microseconds of matrix-core work at most; what it costs elsewhere is a serial
// chain (one workgroup walking the whole of k behind a barrier per step) on a fraction of the compute units.  So here
//   * a workgroup owns a small tile of C (32 x 32 or 64 x 64) and its waves share k between them: wave w takes the 256-element
//     chunks w, w + waves, ... of every plane pair, and the partial sums meet once, in LDS, at the end (one barrier in the
//     whole kernel, two with 64 x 64 tiles);
//   * a wave loads the packed words of its operand rows straight into registers, four words per lane, one chunk ahead of the
//     multiplication.  16-byte loads at any 4-byte alignment; the last piece of a row is read four words from the row's end
//     and the words that an earlier piece has brought already are cleared, so nothing beyond a row is read and K, leading
//     dimensions and channel counts can be anything (of at least four words);
//   * words become E2M1 operands of v_mfma_scale_f32_32x32x64_f8f6f4 in registers.  A +-1 plane: the nibble 0b0010 (1.0) with
//     the sign bit set where the bit is clear.  Two 0/1 planes whose coefficients are c and 2c up to signs: ONE nibble,
//     0.5 (b0 + 2 b1), i.e. one product where the planes one by one would take two.  The planes' powers of two are the block
//     scales of the instruction.  Everything is a multiple of the coefficients' common factor and the sums stay
//     below 2^23 of it (the host checks), so the float accumulation is exact.
//   Phase t of a chunk multiplies bit t of every nibble of a lane's four words (both operands use the same order of k).
#include "qnn_gemm_slice.h"

namespace qnn {

using namespace slice;

namespace {

// BMb x BNb blocks of 32 x 32 per wave; up to kMaxWaves waves share k.
// Waves per SIMD that the registers have to allow: four workgroups with 64 x 64 tiles of single planes, two with pairs of planes (180 to
// 220 registers; held to three they spill: convolutions of 2-bit maps with few tiles are 3 to 8 % slower).
constexpr int waves_per_simd(int ka, int kw, int blocks) { return blocks == 2 && (ka == kPair || kw == kPair) ? 2 : 4; }
template <int kA, int kW, int kRows, int BMb, int BNb, int kMaxWaves>
__global__ __launch_bounds__(64 * kMaxWaves, waves_per_simd(kA, kW, BMb)) void gemm_slice_kernel(const GemmArgs g, const SliceArgs sc, const Tiles tiles) {
    constexpr bool kPixels = kRows != kMatrix;
    constexpr int BM = 32 * BMb, BN = 32 * BNb, kPitch = BN + 4;
    constexpr int NA = kA == kPair ? 2 : 1, NW = kW == kPair ? 2 : 1;  // planes of a digit
    constexpr int ZA = kA == kPair || kA == kMap ? 2 : 1;             // fields of an operand
    // partial sums: a slot per wave; with 64 x 64 tiles half as many (see below), so that four workgroups fit on a compute unit and not two
    // (convolution of a 0/1 map 64 x 56 x 56, 16 -> 32 channels of 5 x 5: 79.3 -> 37.3 us, with the lone plane by itself)
    constexpr uint32_t kSlots = BMb == 2 ? kMaxWaves / 2 : kMaxWaves;
    __shared__ __attribute__((aligned(16))) float part[kSlots][BM][kPitch];
    __shared__ int part_a[kMaxWaves][BM], part_w[kMaxWaves][BN];
    const uint32_t t = threadIdx.x, lane = t & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), waves = blockDim.x >> 6;
    uint32_t tm, tn;
    tile_of_block(blockIdx.x, tiles, tm, tn);
    const uint32_t m0 = tm * BM, n0 = tn * BN;

    // rows of this lane (rows beyond the last repeat it and are not stored)
    uint32_t a_off[BMb], a_in[BMb], w_off[BNb];  // byte offsets from the digit's plane (pixels: of the patch, see patch_of)
#pragma unroll
    for (int b = 0; b < BMb; ++b) {
        uint32_t m = m0 + 32 * b + r;
        m = m < (uint32_t)g.M ? m : (uint32_t)g.M - 1u;
        if constexpr (kPixels) {
            const Patch p = patch_of(g, sc, m, kA == kMap && g.pool_and != nullptr);
            a_off[b] = p.off, a_in[b] = p.in;
        } else {
            a_off[b] = m * (uint32_t)(g.A.ld * 4), a_in[b] = 0u;
        }
    }
#pragma unroll
    for (int b = 0; b < BNb; ++b) {
        uint32_t n = n0 + 32 * b + r;
        n = n < (uint32_t)g.N ? n : (uint32_t)g.N - 1u;
        w_off[b] = n * (uint32_t)(g.ldw * 4);
    }

    // thresholds and flip flags of the epilogue, asked for before the operands
    int32_t threshold = 0;
    uint32_t flip_flag = 0u;
    if (g.epi.T) {
        const uint32_t n = n0 + lane % BN, at = n < (uint32_t)g.N ? n : (uint32_t)g.N - 1u;
        threshold = g.epi.T[at];
        if (g.epi.flip) flip_flag = g.epi.flip[at];
    }

    struct Chunk {
        u32x4 a[NA][BMb], w[NW][BNb];
        uint32_t skip_a[BMb], skip;  // leading words to clear
    };
    const uint8_t *const a_base = reinterpret_cast<const uint8_t *>(g.A.base), *const w_base = reinterpret_cast<const uint8_t *>(g.W);
    auto load = [&](Chunk &x, const SliceDigit &da, const SliceDigit &dw, const uint32_t c) __attribute__((always_inline)) {
        const Piece p = piece_of<kRows>(g, sc, 2u * c + kg);
        x.skip = p.skip;
#pragma unroll
        for (int b = 0; b < BMb; ++b) {
            uint32_t off = a_off[b] + p.off;
            x.skip_a[b] = p.skip;
            if constexpr (kPixels) {
                // outside the image: the plane's first words, cleared before use
                const bool in = ((a_in[b] >> p.ky) & (a_in[b] >> (p.kx + 16u)) & 1u) != 0u;
                off = in ? off : 0u;
                x.skip_a[b] = in ? p.skip : 4u;
            }
            x.a[0][b] = load_piece<kRows>(a_base + da.off0 + off, sc);
            if constexpr (kA == kPair) x.a[1][b] = load_piece<kRows>(a_base + da.off1 + off, sc);
        }
#pragma unroll
        for (int b = 0; b < BNb; ++b) {
            const uint32_t off = w_off[b] + p.w_word * 4u;
            x.w[0][b] = load_piece<kRows>(w_base + dw.off0 + off, sc);
            if constexpr (kW == kPair) x.w[1][b] = load_piece<kRows>(w_base + dw.off1 + off, sc);
        }
    };

    v16f acc[BNb][BMb];
#pragma unroll
    for (int i = 0; i < BNb; ++i)
#pragma unroll
        for (int j = 0; j < BMb; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // row corrections of this lane's words (see make_fields)
    int corr_a[BMb], corr_w[BNb];
#pragma unroll
    for (int b = 0; b < BMb; ++b) corr_a[b] = 0;
#pragma unroll
    for (int b = 0; b < BNb; ++b) corr_w[b] = 0;
    const bool corrected = (kA == kPair || kW == kPair) && sc.corrected != 0;
    // one chunk of one digit pair
    auto multiply = [&](const Chunk &x, const SliceDigit &da, const SliceDigit &dw, const bool clear) __attribute__((always_inline)) {
        u32x4 za[ZA][BMb], zw[NW][BNb];
        auto prepare = [&](auto kind_tag, const u32x4 p0, const u32x4 p1, const SliceDigit &d, const uint32_t skip, const bool clr, u32x4 &z0, u32x4 &z1) __attribute__((always_inline)) {
            if constexpr (decltype(kind_tag)::value == kMap) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = (uint32_t)i >= skip && (kRows != kNarrowPatches || (uint32_t)i < sc.row_words);
                    z0[i] = in ? p0[i] : 0u, z1[i] = in ? 0x22222222u : 0u;
                }
                return 0;
            }
            u32x4 w0 = p0, w1 = p1;
            if (clr) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t keep = (uint32_t)i >= skip ? 0xFFFFFFFFu : 0u;
                    w0[i] &= keep;
                    if constexpr (decltype(kind_tag)::value == kPair) w1[i] &= keep;
                }
            }
            if (sc.modified) apply_inversion<decltype(kind_tag)::value>(d.inv0, d.inv1, d.use1, w0, w1);
            make_fields<decltype(kind_tag)::value>(w0, w1, z0, z1);
            return corrected ? add_sum<decltype(kind_tag)::value>(w0, w1, 0) : 0;
        };
        const int shift = da.lg + dw.lg;
#pragma unroll
        for (int b = 0; b < BMb; ++b) {
            const int sum = prepare(std::integral_constant<int, kA>{}, x.a[0][b], x.a[NA - 1][b], da, x.skip_a[b], clear || kPixels, za[0][b], za[ZA - 1][b]);
            if (corrected) corr_a[b] += ((sum * dw.offset2) << shift) >> 1;
        }
#pragma unroll
        for (int b = 0; b < BNb; ++b) {
            const int sum = prepare(std::integral_constant<int, kW>{}, x.w[0][b], x.w[NW - 1][b], dw, x.skip, kA != kMap && (clear || kPixels), zw[0][b], zw[NW - 1][b]);
            if (corrected) corr_w[b] += ((sum * da.offset2) << shift) >> 1;
        }
        auto phase = [&](auto ph_tag) __attribute__((always_inline)) {
            constexpr int ph = decltype(ph_tag)::value;
            v4i fa[BMb], fw[BNb];
#pragma unroll
            for (int b = 0; b < BMb; ++b) fa[b] = make_operand<kA>(za[0][b], za[ZA - 1][b], ph);
#pragma unroll
            for (int b = 0; b < BNb; ++b) fw[b] = make_operand<kW>(zw[0][b], zw[NW - 1][b], ph);
#pragma unroll
            for (int i = 0; i < BNb; ++i)
#pragma unroll
                for (int j = 0; j < BMb; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(fw[i]), widen(fa[j]), acc[i][j], 4, 4, ph, dw.scale, ph, da.scale);
        };
        phase(std::integral_constant<int, 0>{});
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
    };

    // this wave's items: (digit pair, chunk) number wave, wave + waves, ... with the chunks innermost
    const uint32_t pairs = (uint32_t)(sc.a.count * sc.w.count);
    // waves that have an item (workgroups of more than four waves are made no larger)
    const uint32_t parts = kMaxWaves > 4 || pairs * sc.chunks > waves ? waves : pairs * sc.chunks;
    uint32_t pair = 0, c = wave, ia = 0, iw = 0;  // pair ia * (digits of the right operand) + iw
    auto settle = [&]() __attribute__((always_inline)) {
        while (c >= sc.chunks && pair < pairs) {
            c -= sc.chunks, ++pair;
            if (++iw == (uint32_t)sc.w.count) iw = 0, ++ia;
        }
    };
    settle();
    Chunk cur, nxt;
    if (pair < pairs) load(cur, sc.a.d[ia], sc.w.d[iw], c);
    while (pair < pairs) {
        const uint32_t c_now = c, ia_now = ia, iw_now = iw;
        c += waves;
        settle();
        if (pair < pairs) load(nxt, sc.a.d[ia], sc.w.d[iw], c);
        const bool clear = !kPixels && 8u * c_now + 8u > sc.row_words;
        multiply(cur, sc.a.d[ia_now], sc.w.d[iw_now], clear);
        cur = nxt;
    }

    // partial sums to LDS: register v of block [i][j] is C[m][n], m = 32 j + lane mod 32, n = 32 i + 8 (v / 4) + 4 kg + v mod 4
    auto slot_of = [&](const uint32_t slot, const int i, const int j, const int q) __attribute__((always_inline)) {
        return reinterpret_cast<f32x4 *>(&part[slot][32 * j + r][32 * i + 8 * q + 4 * kg]);
    };
    auto put = [&](const uint32_t slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < BNb; ++i)
#pragma unroll
            for (int j = 0; j < BMb; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) *slot_of(slot, i, j, q) = f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    };
    if (kSlots < kMaxWaves && parts > kSlots) {
        // the upper half of the waves leaves its sums to the lower half, each wave of which adds those of one slot to its own
        if (wave >= kSlots && wave < parts) put(wave - kSlots);
        __syncthreads();
        if (wave + kSlots < parts) {
#pragma unroll
            for (int i = 0; i < BNb; ++i)
#pragma unroll
                for (int j = 0; j < BMb; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = *slot_of(wave, i, j, q);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
                    }
        }
    }
    const uint32_t slots = parts < kSlots ? parts : kSlots;
    if (wave < slots) put(wave);
    if (corrected && wave < parts) {
#pragma unroll
        for (int b = 0; b < BMb; ++b) {
            const int v = corr_a[b] + __shfl_xor(corr_a[b], 32, 64);
            if (kg == 0) part_a[wave][32 * b + r] = v;
        }
#pragma unroll
        for (int b = 0; b < BNb; ++b) {
            const int v = corr_w[b] + __shfl_xor(corr_w[b], 32, 64);
            if (kg == 0) part_w[wave][32 * b + r] = v;
        }
    }
    __syncthreads();
    const uint32_t rows = (uint32_t)g.M - m0 < (uint32_t)BM ? (uint32_t)g.M - m0 : (uint32_t)BM;
    if (!g.epi.T) {
        const bool vec = (g.epi.ldc % 4 == 0) && (reinterpret_cast<uintptr_t>(g.epi.C) % 16 == 0);
        for (uint32_t i = t; i < rows * (BN / 4); i += blockDim.x) {
            const uint32_t row = i / (BN / 4), col = 4u * (i % (BN / 4));
            f32x4 s = *reinterpret_cast<const f32x4 *>(&part[0][row][col]);
            for (uint32_t w = 1; w < slots; ++w) s += *reinterpret_cast<const f32x4 *>(&part[w][row][col]);
            int corr[4] = {0, 0, 0, 0};
            if (corrected)
                for (uint32_t w = 0; w < parts; ++w)
#pragma unroll
                    for (int e = 0; e < 4; ++e) corr[e] += part_a[w][row] + part_w[w][col + e];
            i32x4 val;
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = (int32_t)((uint32_t)((int32_t)s[e] - corr[e]) * sc.alpha + sc.c0);
            const int64_t n = (int64_t)n0 + col;
            int32_t *dst = g.epi.C + (int64_t)(m0 + row) * g.epi.ldc + n;
            if (vec && n + 4 <= g.N)
                __builtin_nontemporal_store(val, reinterpret_cast<i32x4 *>(dst));
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < g.N) dst[e] = val[e];
        }
    } else {
        // a lane keeps its column; a ballot packs 64 columns of a row (or 32 of each of two rows)
        constexpr uint32_t kRowsPerWave = 64 / BN;
        const uint32_t col = lane % BN;
        const int64_t n = (int64_t)n0 + col;
        const bool live = n < g.N;
        const int32_t T = threshold;
        const bool flip = live && flip_flag != 0u;
        if constexpr (kA == kMap && BN == 32) {
            // four rows are a pixel behind the pooling: OR, or AND where the filter's bits are flipped
            if (g.pool_and) {
                const uint32_t all = (g.pool_and[tn] ^ g.pool_invert);
                for (uint32_t row0 = 4u * wave; row0 < rows; row0 += 4u * waves) {
                    uint64_t bits[2];
#pragma unroll
                    for (uint32_t h = 0; h < 2; ++h) {
                        const uint32_t row = row0 + 2u * h + kg;
                        float s = part[0][row][col];
                        for (uint32_t w = 1; w < slots; ++w) s += part[w][row][col];
                        bits[h] = __ballot(live && (((int32_t)s >= T) != flip));
                    }
                    const uint32_t a = (uint32_t)bits[0], b = (uint32_t)(bits[0] >> 32), c = (uint32_t)bits[1], d = (uint32_t)(bits[1] >> 32);
                    if (lane == 0u) g.epi.out_bits[(int64_t)((m0 + row0) >> 2) * g.epi.ldo + tn] = ((a | b | c | d) & ~all) | (a & b & c & d & all);
                }
                return;
            }
        }
        for (uint32_t row0 = wave * kRowsPerWave; row0 < rows; row0 += waves * kRowsPerWave) {
            const uint32_t row = row0 + lane / BN;  // (below BM: BM is a multiple of kRowsPerWave)
            float s = part[0][row][col];
            for (uint32_t w = 1; w < slots; ++w) s += part[w][row][col];
            int corr = 0;
            if (corrected)
                for (uint32_t w = 0; w < parts; ++w) corr += part_a[w][row] + part_w[w][col];
            const int32_t val = (int32_t)((uint32_t)((int32_t)s - corr) * sc.alpha + sc.c0);
            const unsigned long long bits = __ballot(live && ((val >= T) != flip));
            const int64_t n_word = (int64_t)n0 + (BN == 64 ? (lane & 32u) : 0u);
            if ((lane & 31u) == 0u && row < rows && n_word < g.N)
                g.epi.out_bits[(int64_t)(m0 + row) * g.epi.ldo + n_word / 32] = (uint32_t)(bits >> lane);
        }
    }
}

// The digits of an operand; false if a coefficient is not the common factor times a power of two, or offsets leave 32 bits.
// bits: a +-1 plane as 0 / 1; one: a lone 0 / 1 plane by itself and not as half of a pair.
bool make_digits(const Planes &pl, int64_t plane_stride, bool bits, bool one, SliceOperand &op, int &kind, int64_t &gcd_out, int64_t &sum_abs_over_gcd) {
    std::memset(&op, 0, sizeof(op));
    int64_t gcd = 0;
    for (int p = 0; p < pl.count; ++p) {
        int64_t x = gcd, y = pl.coef[p] < 0 ? -(int64_t)pl.coef[p] : pl.coef[p];
        if (y == 0) return false;
        while (y) {
            const int64_t r = x % y;
            x = y, y = r;
        }
        gcd = x;
    }
    if (pl.count == 1 && pl.coef[0] < 0) gcd = -gcd;  // one plane: the sign goes into the factor
    int order[QNN_MAX_PLANES], lg[QNN_MAX_PLANES];
    int64_t d[QNN_MAX_PLANES], sum = 0;
    for (int p = 0; p < pl.count; ++p) {
        d[p] = pl.coef[p] / gcd;
        const int64_t ad = d[p] < 0 ? -d[p] : d[p];
        if (ad > (1 << 20) || (ad & (ad - 1))) return false;
        lg[p] = 0;
        while (((int64_t)1 << lg[p]) < ad) ++lg[p];
        sum += ad;
        if (4.0L * (long double)p * (long double)plane_stride >= 4294967296.0L) return false;
        int i = p;
        for (; i > 0 && lg[order[i - 1]] > lg[p]; --i) order[i] = order[i - 1];
        order[i] = p;
    }
    const bool sign = pl.mode == QNN_PLANE_SIGN;
    kind = sign ? (bits ? kOne : kPm1) : (one && pl.count == 1 ? kOne : kPair);
    for (int i = 0; i < pl.count; ++i) {
        SliceDigit &e = op.d[op.count++];
        const int p = order[i];
        e.off0 = e.off1 = (uint32_t)((int64_t)p * plane_stride * 4);
        e.lg = lg[p] + (sign && bits ? 1 : 0);
        e.inv0 = d[p] < 0 ? 0xFFFFFFFFu : 0u;
        if (kind == kPair && i + 1 < pl.count && lg[order[i + 1]] == lg[p] + 1) {
            const int p1 = order[++i];
            e.off1 = (uint32_t)((int64_t)p1 * plane_stride * 4);
            e.use1 = 0xFFFFFFFFu;
            e.inv1 = d[p1] < 0 ? 0xFFFFFFFFu : 0u;
            e.offset2 = d[p1] < 0 ? 4 : 0;
        }
        if (sign)
            e.offset2 = bits ? 1 : 0;
        else
            e.offset2 += d[p] < 0 ? 2 : 0;
        // a set first bit is worth 1 (kPm1), 0.5 (kPair), 0.5 / 1 / 2 / 1 in phases 0 .. 3 (kOne) as an operand; the factor 2 of a +-1
        // plane multiplied as 0 / 1 is left to the epilogue (alpha_sum), so that |S| has the bound of the values' sums
        const int one = 127 + lg[p];
        e.scale = kind == kPm1 ? one * 0x01010101 : (kind == kPair ? (one + 1) * 0x01010101 : one * 0x01010101 + 1 - 0x10000);
    }
    gcd_out = gcd, sum_abs_over_gcd = sum;
    return true;
}

uint32_t magic(int64_t d) { return (uint32_t)((4294967296LL + d - 1) / d); }  // d >= 2

}  // namespace

namespace slice {
bool slice_args(const GemmArgs &g, bool bits, SliceArgs &sc, int &kind_a, int &kind_w) {
    std::memset(&sc, 0, sizeof(sc));
    if (g.A.rows_are_bytes) return false;
    const bool pix = g.A.rows_are_pixels != 0;
    int64_t ga, gw, sa, sw;
    if (!make_digits(g.pa, g.A.plane_stride, bits, true, sc.a, kind_a, ga, sa) || !make_digits(g.pw, g.strideW, bits, bits, sc.w, kind_w, gw, sw)) return false;
    const int64_t row_words = pix ? g.A.Cw : g.Kw;
    if (row_words < (pix ? 1 : 4)) return false;
    if (pix && (g.A.KH > 15 || g.A.KW > 15)) return false;  // (which taps lie inside the image: sixteen bits each way, one spare)
    const int64_t ppt = ceil_div(row_words, 4), taps = pix ? (int64_t)g.A.KH * g.A.KW : 1, pieces = ppt * taps;
    if (pieces >= 32768 || taps >= 32768) return false;  // (the quotients by multiplication are exact below 2^32 / divisor)
    sc.row_words = (uint32_t)row_words, sc.ppt = (uint32_t)ppt, sc.taps = (uint32_t)taps;
    sc.magic_ppt = ppt > 1 ? magic(ppt) : 0u, sc.magic_kw = pix && g.A.KW > 1 ? magic(g.A.KW) : 0u;
    sc.chunks = (uint32_t)ceil_div(pieces, 2);
    if (pix) {
        if ((int64_t)g.A.Ho * g.A.Wo > 0x7FFFFFFFLL) return false;
        sc.inv_hw = inverse_of((int64_t)g.A.Ho * g.A.Wo), sc.inv_w = inverse_of(g.A.Wo);
    }
    // |S| in units of the common factors stays below 2^23: exact float sums, and with |alpha_sum| below 2^23 a 24-bit product in the
    // tiled kernel's epilogue.  (The same conditions whether or not +-1 planes enter as 0 / 1: what one kernel takes the other takes.)
    if ((long double)sa * (long double)sw * 256.0L * sc.chunks >= 8388608.0L) return false;
    const int64_t twice = (g.pa.mode == QNN_PLANE_SIGN ? 2 : 1) * (g.pw.mode == QNN_PLANE_SIGN ? 2 : 1);
    if (ga * gw * twice >= 8388608 || ga * gw * twice <= -8388608) return false;
    // 32-bit byte offsets
    const long double a_words = pix ? (long double)g.M / ((long double)g.A.Ho * g.A.Wo) * g.A.H * g.A.Wd * g.A.Cw : (long double)g.M * g.A.ld;
    if (4.0L * a_words >= 4294967296.0L || 4.0L * (long double)g.N * g.ldw >= 4294967296.0L) return false;
    if (g.M > 0x7FFFFF00LL || g.N > 0x7FFFFF00LL) return false;
    sc.alpha = (uint32_t)(ga * gw);
    sc.alpha_sum = (uint32_t)(ga * gw * (bits ? twice : 1));
    // offsets of the digits (see make_fields): the constant part, over every processed element
    int64_t constant = 0;
    for (int i = 0; i < sc.a.count; ++i)
        for (int j = 0; j < sc.w.count; ++j) {
            const SliceDigit &da = sc.a.d[i], &dw = sc.w.d[j];
            constant += ((int64_t)da.offset2 * dw.offset2 * 64 * sc.chunks) << (da.lg + dw.lg);
            if (dw.offset2) sc.sum_a = sc.corrected = 1;
            if (da.offset2) sc.sum_w = sc.corrected = 1;
            if (da.inv0 || da.inv1 || dw.inv0 || dw.inv1 || (kind_a == kPair && !da.use1) || (kind_w == kPair && !dw.use1)) sc.modified = 1;
        }
    sc.c0 = (uint32_t)constant * sc.alpha;
    sc.clear_w = g.pa.mode == QNN_PLANE_SIGN;
    sc.ragged = row_words % 4 != 0;
    // +-1 planes on both sides: a processed element beyond K is (-sum coefA)(-sum coefW) instead of 0
    if (g.pa.mode == QNN_PLANE_SIGN && g.pw.mode == QNN_PLANE_SIGN) {
        int64_t ca = 0, cw = 0;
        for (int p = 0; p < g.pa.count; ++p) ca += g.pa.coef[p];
        for (int p = 0; p < g.pw.count; ++p) cw += g.pw.coef[p];
        const int64_t surplus = 256 * (int64_t)sc.chunks - g.K;
        sc.c0 += (uint32_t)(-surplus * ca * cw);
    }
    return true;
}
}  // namespace slice

namespace {

typedef void (*SliceFn)(const GemmArgs, const SliceArgs, const Tiles);
template <int kRows, int BMb, int BNb, int kMaxWaves>
SliceFn slice_kernel(int ka, int kw) {
    if (ka == kPm1) return kw == kPm1 ? gemm_slice_kernel<kPm1, kPm1, kRows, BMb, BNb, kMaxWaves> : gemm_slice_kernel<kPm1, kPair, kRows, BMb, BNb, kMaxWaves>;
    if (ka == kOne) return kw == kPm1 ? gemm_slice_kernel<kOne, kPm1, kRows, BMb, BNb, kMaxWaves> : gemm_slice_kernel<kOne, kPair, kRows, BMb, BNb, kMaxWaves>;
    return kw == kPm1 ? gemm_slice_kernel<kPair, kPm1, kRows, BMb, BNb, kMaxWaves> : gemm_slice_kernel<kPair, kPair, kRows, BMb, BNb, kMaxWaves>;
}
template <int kRows>
SliceFn slice_kernel(int ka, int kw, bool large, bool four) {
    if (large) return slice_kernel<kRows, 2, 2, 4>(ka, kw);
    return four ? slice_kernel<kRows, 1, 1, 4>(ka, kw) : slice_kernel<kRows, 1, 1, 16>(ka, kw);
}

}  // namespace

// About how long a product takes on the tiled kernel (microseconds): a pair of digits costs a latency per element of k and, for each
// tile of a compute unit, the making of its operands (375 products of 1 to 16 pairs within 7 % as a rule, at most 22).  Below 192 tiles,
// which go to smaller ones, a rough figure (1024 x 1024 x 8192: 49 and 29 for 4 x 4 and 4 x 1 planes, measured 50 and 20).
static double tile_us(const GemmArgs &g, const SliceArgs &sc, int ka, int kw) {
    const int pairs_of_planes = (ka == kPair ? 1 : 0) + (kw == kPair ? 1 : 0);
    constexpr double kLatency[3] = {0.9e-3, 1.2e-3, 0.9e-3}, kTile[3] = {1.3e-3, 1.6e-3, 2.0e-3}, kStore[3] = {0.53e-6, 0.53e-6, 0.76e-6};
    const int64_t tiles = ceil_div(g.M, 128) * ceil_div(g.N, 128);
    const double tiles_each = tiles < 192 ? (double)tiles / compute_units() : (double)ceil_div(tiles, compute_units());
    const double k = 256.0 * sc.chunks * sc.a.count * sc.w.count;
    return 2.8 + k * (kLatency[pairs_of_planes] + kTile[pairs_of_planes] * tiles_each) + kStore[pairs_of_planes] * (double)g.M * (double)g.N;
}

// 32 x 32 tiles: four waves each or sixteen (see launch_gemm_slice)
static bool four_waves(int64_t items, int64_t tiles) { return items <= 4 || (tiles > 512 && (tiles > 1024 || items <= 32)); }

// The same on the tiles that take over below 192, 64 x 64 or 32 x 32 (220 products of five to eight planes and a +-1 plane, 64 to 30000
// rows and columns, 256 to 20000 elements of k: within 15 % as a rule, at most 23).
static double small_tile_us(const GemmArgs &g, const SliceArgs &sc) {
    const double cus = compute_units(), elements = (double)g.M * (double)g.N;
    const int64_t items = (int64_t)sc.chunks * sc.a.count * sc.w.count, tiles64 = ceil_div(g.M, 64) * ceil_div(g.N, 64), tiles32 = ceil_div(g.M, 32) * ceil_div(g.N, 32);
    const double k = 256.0 * (double)items;
    if (tiles64 >= 160 && g.M > 32 && g.N > 32)
        return 4.0 + k * (0.44e-3 + 0.23e-3 * (double)tiles64 / cus + 0.57e-3 * (double)ceil_div(tiles64, compute_units())) + 2.3e-6 * elements;
    if (four_waves(items, tiles32)) return 4.0 + 0.535e-3 * k * (double)tiles32 / cus;
    return 4.0 + k * (0.063e-3 * (double)tiles32 / cus + 0.307e-3 * (double)ceil_div(tiles32, compute_units())) + 2.7e-6 * elements;
}

// (For the choice against another way of the backward step, whose other launches take longer than it assumes: a quarter is added to the small
// tiles' time, and tile_us's rough figure stays where it is the smaller.)
double slice_us(const GemmArgs &g) {
    SliceArgs sc;
    int ka, kw;
    if (!slice_args(g, false, sc, ka, kw)) return 1e30;
    const double tiled = tile_us(g, sc, ka, kw);
    if (ceil_div(g.M, 128) * ceil_div(g.N, 128) >= 192 && g.M >= 96 && g.N >= 96) return tiled;
    const double small = 1.25 * small_tile_us(g, sc);
    return small < tiled ? small : tiled;
}

// Where the library's own choice goes to these kernels.  Measured (us, GPU time; route of the shape -> best of these; numbers of tiles are
// counts for 256 compute units):
//   vector-ALU route: everything (32 x 4096 x 4096 20 -> 4.5; 20 x 4096 x 2048 with 4 x 4 planes 134 -> 8; convolution of four
//     13 x 13 maps, 384 -> 256 channels, 39 -> 5; 1000 x 1000 x 1000 8.7 -> 5.3);
//   single planes that the panel-fed kernel does not take or rows below 512 elements: everything (1999 x 3001 x 2500 82 -> 21);
//   other single planes, int32 sums: while 64 x 64 tiles make one round at most (256 x 1024 x 8192 24 -> 6; 10000 x 256 x 8192, 628
//     tiles, 25 -> 19; 2048^3, 1024, 12.8 -> 11.2), and while the panels' 256 x 128 tiles leave compute units idle and rows are short
//     (3000 x 2048, 192 such tiles, x 1024 11.2 -> 9.7, x 2048 13.4 and 13.7, x 4096 18.0 against 19.7, x 8192 26.8 against 32.5);
//   int32 sums of rows that are no whole groups of 1024 (447 products of 160 to 2600 tiles of 128 x 128, t, rows of 512 to 7000; here / panels):
//     C in 16-byte pieces: while its 64 x 64 tiles make one round here, five a compute unit (t <= 320 .66 to 1.05, beyond 1.04 to 1.4);
//     C word by word, which takes the panels longer where their tiles do not make one round, two a unit: while 64 x 64 tiles are at most three a
//       unit (t <= 200 .87 to 1.0, 216 to 512 1.02 to 1.2), or four where ragged edges make more than one 128 x 128 tile of them a unit (2502 x
//       1573 x 3584, t = 260, .87), and beyond one round with short rows: t up to 1024, where 128 x 256 tiles make one,
//       K < 1400 (516 x 673 .90, 759 x 1406 .99, 854 x 2993 1.1), just behind it (t = 1026 to 1280) K < 4000 (.82 to .96, K above 4800 1.0), from there on
//       K < 2500 (.82 to 1.03, above 1.02 to 1.16).
//     With C's lines in no cache (six outputs in turn, 350 MB) the panels fall back by up to a third more beyond t = 900: their parts of a
//       line arrive further apart.
//   the same with threshold output, which costs the panel-fed kernel less: while 64 x 64 tiles are few (512 x 4096 x 4096, 512 tiles, 14.7
//     -> 11.4; 10000 x 256 x 2048, 628, 10.4 -> 10.3; 1500 x 2048 x 2048, 768, 10.6 against 11.2; 20000 x 256 x 4096, 1252, 15.0 against
//     21.0);
//   several planes that the kernels with merged planes take: everything that makes no 192 tiles of 128 x 128 (1024 x 1024 x 8192 with 4 x 4
//     planes 81 -> 50; 1000 x 1000 x 16384 144 -> 100), and by the expected times else: the tiled kernel's time grows with the pairs of
//     digits, that of merged planes does not (4096^3 with 4, 5, 7 planes x 1: 69, 101, 129 on tiles, 77 merged; 2240 x 4096 x 2048: 28,
//     39, 51 and 42; 2 x 2 and 4 x 4 planes: 25, 62 and 42).  Of 375 products on both sides the choice cost 0.3 % of the time, at most 15 %.
bool slice_preferred(const GemmArgs &g, int route) {
    SliceArgs sc;
    int ka, kw;
    if (!slice_args(g, false, sc, ka, kw)) return false;
    if (route == QNN_ENGINE_MFMA_FP4 && panel_takes(g)) {
        const int64_t tiles64 = ceil_div(g.M, 64) * ceil_div(g.N, 64);
        if (g.epi.T) return tiles64 <= (g.N < 512 || g.K > 4096 ? 640 : 288);
        const bool whole = g.Kw % 32 == 0 && g.A.ld % 4 == 0 && g.ldw % 4 == 0 && (reinterpret_cast<uintptr_t>(g.A.base) | reinterpret_cast<uintptr_t>(g.W)) % 16 == 0;
        if (!whole) {
            const int64_t cus = compute_units(), tiles = ceil_div(g.M, 128) * ceil_div(g.N, 128);
            const bool words = g.epi.ldc % 4 != 0 || reinterpret_cast<uintptr_t>(g.epi.C) % 16 != 0;  // C leaves word by word
            if (!words) return tiles64 <= 5 * cus;
            if (tiles64 <= (tiles > cus ? 4 : 3) * cus) return true;
            return tiles > 2 * cus && g.K < (tiles <= 4 * cus ? 1400 : (tiles <= 5 * cus ? 4000 : 2500));
        }
        return tiles64 <= 1024 || (g.K <= 2048 && ceil_div(g.M, 256) * ceil_div(g.N, 128) < 256);
    }
    if (route == QNN_ENGINE_MFMA_LDS && ceil_div(g.M, 128) * ceil_div(g.N, 128) >= 192) return tile_us(g, sc, ka, kw) <= stage_us(g);
    return true;
}

int launch_gemm_slice(const GemmArgs &g, hipStream_t s) {
    SliceArgs sc;
    int ka, kw;
    if (!slice_args(g, false, sc, ka, kw)) return fail(QNN_ERR_UNSUPPORTED, "sliced matrix-core kernel cannot take these arguments");
    const bool pix = g.A.rows_are_pixels != 0;
    // Tile by the number of tiles (the lines are counts for 256 compute units): 128 x 128 where there are enough of them for the chip
    // (1024 x 1024 x 4096, 64 tiles, 13.3 us against 7.7 with 64 x 64; convolutions pay more per group of k: from 384 tiles on), 32 x 32
    // with k shared by up to sixteen waves where 64 x 64 tiles are few (256 x 1024 x 8192, 64 tiles, 5.9 against 9.6 us; 1000 x 1000 x
    // 1000, 256 tiles, 5.8 against 5.2) or mostly padding.
    // Single planes on both sides: four workgroups with 64 x 64 tiles share a compute unit, and while about one round of them is all
    // there is they beat the larger tiles (GPU time, 128 x 128 -> 64 x 64: 1800 x 1800 x 500, 841 tiles, 9.8 -> 6.5 us, x 4000 17.9 -> 14.0;
    // 40000 x 96 x 256, 1250 tiles, 11.2 -> 8.0; 1999 x 3001 x 2048, 1504 tiles, 18.2 -> 19.4), with threshold output only while k is
    // short (1800 x 1800 x 500 7.5 -> 6.7, x 2048 11.0 -> 11.5).
    const int64_t items = (int64_t)sc.chunks * sc.a.count * sc.w.count, tiles64 = ceil_div(g.M, 64) * ceil_div(g.N, 64);
    const bool one_round = ka != kPair && kw != kPair && (g.epi.T ? tiles64 <= 1024 && items <= 2 : tiles64 <= 1280);
    if (!one_round && ceil_div(g.M, 128) * ceil_div(g.N, 128) >= (pix ? 384 : 192) && g.M >= 96 && g.N >= 96) return launch_gemm_tile(g, s);
    const bool large = tiles64 >= 160 && g.M > 32 && g.N > 32;
    const int64_t edge = large ? 64 : 32, tiles_m = ceil_div(g.M, edge), tiles_n = ceil_div(g.N, edge), tiles = tiles_m * tiles_n;
    if (tiles > 0x7FFFFFFFLL) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
    // 32 x 32 tiles: four waves each where there are more tiles than workgroups of sixteen waves fit on the chip (100000 x 10 x 4096 25.6
    // -> 17.6 us, 32768 outputs of 20 rows x 4096 with 4 x 4 planes 43.8 -> 34.3), unless the rows are long and the tiles not much more
    // than that (20000 x 10 x 16384 17.0 against 18.5).  Never fewer than four: waves without a chunk of k still share the epilogue
    // (64 x 64 tiles, 1000 x 1000 x 128: 7.1 -> 4.8 us).
    const bool four = large || four_waves(items, tiles);
    const int waves = four ? 4 : (items < 16 ? (int)items : 16);
    const SliceFn fn = !pix ? slice_kernel<kMatrix>(ka, kw, large, four) : (g.A.Cw < 4 ? slice_kernel<kNarrowPatches>(ka, kw, large, four) : slice_kernel<kPatches>(ka, kw, large, four));
    return QNN_LAUNCH("gemm_slice", fn, dim3((unsigned)tiles), dim3(64u * waves), 0, s, g, sc, make_tiles(tiles_m, tiles_n));
}

// The same kernel on a +-1 map's plane "value is -1" (3 x 3 convolution, channels that fill whole words): half the loads and two thirds of the
// instructions of the 2-bit code, no plane "inside the image" to fill, and 2 x 2 pooling in the epilogue.  Bound: latency.  Where 32 x 32 tiles are
// taken.  App. A ConvNet of width 128, 4 images of 32 x 32, all layers: 56 -> 45 us with all five convolutions here (12 -> 9
// launches); 1 image of 16 x 16 46.4 -> 38.6.
namespace slice {
static bool map_args(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N, bool pooled, GemmArgs &g, SliceArgs &sc) {
    const int64_t Cw = words_for(C);
    if (B < 1 || H < 1 || Wd < 1 || H > 32767 || Wd > 32767 || C % 32 != 0 || C > (1 << 24) || N < 1 || (pooled && (H < 2 || Wd < 2))) return false;
    if (B > 0x7FFFFF00LL / (H * Wd)) return false;
    const int64_t tiles64 = ceil_div(B * H * Wd, 64) * ceil_div(N, 64);
    if (tiles64 >= 160 && B * H * Wd > 32 && N > 32) return false;
    std::memset(&g, 0, sizeof(g));
    g.A.rows_are_pixels = 1;
    g.A.H = (int)H, g.A.Wd = (int)Wd, g.A.Ho = (int)H, g.A.Wo = (int)Wd, g.A.Cw = (int)Cw, g.A.KH = 3, g.A.KW = 3, g.A.pad = 1, g.A.stride = 1;
    g.pa.count = 1, g.pa.mode = QNN_PLANE_SIGN, g.pa.coef[0] = 1;
    g.pw.count = 1, g.pw.mode = QNN_PLANE_SIGN, g.pw.coef[0] = 1;
    g.ldw = g.Kw = 9 * Cw;
    g.M = B * H * Wd, g.N = N, g.K = 9 * C;
    int ka, kw;
    if (!slice_args(g, false, sc, ka, kw)) return false;
    sc.c0 = 0;  // (elements beyond a row are zeros here)
    if (pooled) {
        g.A.Ho = (int)(H / 2), g.A.Wo = (int)(Wd / 2);
        g.M = 4 * B * g.A.Ho * g.A.Wo;
        sc.inv_hw = inverse_of((int64_t)g.A.Ho * g.A.Wo), sc.inv_w = inverse_of(g.A.Wo);
    }
    return true;
}

bool map_supports(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N, bool pooled) {
    GemmArgs g;
    SliceArgs sc;
    return map_args(B, H, Wd, C, N, pooled, g, sc);
}

int launch_map(const uint32_t *plane, int64_t B, int H, int Wd, int64_t C, const uint32_t *W, int64_t N, const int32_t *T, const uint8_t *flip, uint32_t *out,
               int64_t ldo, const uint32_t *pool_and, bool pool_invert, hipStream_t s) {
    GemmArgs g;
    SliceArgs sc;
    if (!map_args(B, H, Wd, C, N, pool_and != nullptr, g, sc)) return fail(QNN_ERR_UNSUPPORTED, "convolution of a +-1 map: shape not supported");
    g.A.base = plane, g.W = W;
    g.epi.T = T, g.epi.flip = flip, g.epi.out_bits = out, g.epi.ldo = ldo;
    g.pool_and = pool_and, g.pool_invert = pool_invert ? 0xFFFFFFFFu : 0u;
    const int64_t tiles_m = ceil_div(g.M, 32), tiles_n = ceil_div(N, 32), tiles = tiles_m * tiles_n, items = sc.chunks;
    if (tiles > 0x7FFFFFFFLL) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
    const bool four = four_waves(items, tiles), narrow = g.A.Cw < 4;
    const SliceFn fn = narrow ? (four ? gemm_slice_kernel<kMap, kPm1, kNarrowPatches, 1, 1, 4> : gemm_slice_kernel<kMap, kPm1, kNarrowPatches, 1, 1, 16>)
                              : (four ? gemm_slice_kernel<kMap, kPm1, kPatches, 1, 1, 4> : gemm_slice_kernel<kMap, kPm1, kPatches, 1, 1, 16>);
    return QNN_LAUNCH("gemm_slice", fn, dim3((unsigned)tiles), dim3(64u * (four ? 4 : (items < 16 ? (int)items : 16))), 0, s, g, sc, make_tiles(tiles_m, tiles_n));
}
}  // namespace slice

}  // namespace qnn
