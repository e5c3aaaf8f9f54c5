// Matrix-core kernel for products of ordinary size whose rows can be anything: odd widths, rows that start at any word,
// several bit planes, convolutions (the larger sibling of qnn_gemm_slice.hip; same digits, same operands).
//
// Bound: the vector instructions that make the operands, 13 to 19 per matrix-core instruction by the counters (about twice the
// matrix cores' time), and the waits between them.  A workgroup of four waves owns a 128 x 128 tile of C, a wave 64 x 64 of it (2 x 2
// blocks, so that an operand feeds two products); three workgroups share a compute unit (two where both operands have two planes) and
// fill each other's waits.  2-bit convolution 256 x 13 x 13, 384 -> 256 channels: 62.6 -> 26.9 us against planes merged to bytes in LDS.
// (Single planes of 512 elements and more go to qnn_gemm_panel_kernel.h, whose loads write LDS by themselves: 1999 x 3001 x 2500 19.9 ->
// 17.2 us.)
//   * Loads: a wave reads sixteen rows x 64 contiguous bytes, or eight x 128, per instruction (an instruction whose 64 lanes read
//     64 rows costs the address path of the compute unit 64 cycles, eight rows 16 to 19), 16 bytes per lane at any 4-byte
//     alignment, a group ahead of the multiplication, into registers.  A group is four pieces of a row: of eight, the loads in
//     flight take the registers of the third workgroup, and that costs more than half as many barriers give (GPU time, eight ->
//     four pieces: 2-bit convolution 256 x 13 x 13, 384 -> 256 channels, 34.1 -> 27.8 us, 4-bit 54.3 -> 46.3; products
//     3000 x 4096 x 3000 23.8 -> 21.9).  It is eight where that brings no third workgroup or takes none away: matrices of
//     two planes a digit on both sides (1000 x 4096 x 2048 of 4 bits: 30.4 us against 32.8 with four).
//     The last piece of a row is read four words from its end and the words an earlier piece has brought are cleared, so nothing
//     beyond a row is read.
//   * The words go to LDS once per workgroup, already cleared and, for two planes of a digit, already interleaved; piece c of row
//     r sits at piece c xor (r / 2 mod 8), r / 4 mod 4 in groups of four, so that writes (whole rows of a group) and reads (32
//     rows, one piece) use all banks.
//   * Epilogue through LDS: a 32 x 64 block per wave at a time, so that C leaves as 256-byte pieces of rows.
#include "qnn_gemm_panel_kernel.h"
#include "qnn_gemm_slice.h"

namespace qnn {

using namespace slice;

namespace {

constexpr int kTileThreads = 256;
constexpr int kTile = 128;
constexpr int kStagePitch = 68;  // floats per row of the epilogue's block: 64 and a gap

// (a wave's LDS operations execute in order: only the compiler has to be kept from reordering them)
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int kA, int kW, int kRows>
__global__ __launch_bounds__(kTileThreads, kA == kPair && kW == kPair ? 2 : 3) void gemm_tile_kernel(const GemmArgs g, const SliceArgs sc, const Tiles tiles) {
    constexpr bool kPixels = kRows != kMatrix;
    constexpr int NA = kA == kPair ? 2 : 1, NW = kW == kPair ? 2 : 1;  // planes of a digit
    // 16-byte pieces of a row per group (two of them make a chunk of 256 elements)
    constexpr int kPieces = kA == kPair && kW == kPair && !kPixels ? 8 : 4;
    constexpr int kRowBytes = 16 * kPieces, kPlaneBytes = kTile * kRowBytes;    // a group of one plane of an operand
    constexpr int kLoads = kPieces / 2, kLoadRows = kTile / kLoads;            // per plane: loads of a wave, rows of a load of the workgroup
    constexpr uint32_t kSwizzle = kPieces == 8 ? 1 : 2;                        // rows of this power of two share an order of pieces
    constexpr int kOperandBytes = (NA + NW) * kPlaneBytes, kEpiBytes = 4 * 32 * kStagePitch * 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kOperandBytes > kEpiBytes ? kOperandBytes : kEpiBytes];
    __shared__ __attribute__((aligned(16))) int corr_a[kTile], corr_w[kTile];  // row corrections (see make_fields)
    const uint32_t t = threadIdx.x, lane = t & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 1, wn = wave & 1u;
    uint32_t tm, tn;
    tile_of_block(blockIdx.x, tiles, tm, tn);
    const uint32_t m0 = tm * kTile, n0 = tn * kTile;

    // ------------------------------------------------------------------------------------------------ loads
    // load i of a plane: piece lane mod kPieces of rows kLoadRows i + prow
    const uint32_t prow = (uint32_t)(64 / kPieces) * wave + lane / kPieces, piece0 = lane % kPieces;
    uint32_t a_off[kLoads], a_in[kLoads], w_off[kLoads];  // byte offset of the row (pixels: of the patch, see patch_of)
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        uint32_t m = m0 + kLoadRows * i + prow;
        m = m < (uint32_t)g.M ? m : (uint32_t)g.M - 1u;  // (rows beyond the last repeat it and are not stored)
        if constexpr (kPixels) {
            const Patch p = patch_of(g, sc, m);
            a_off[i] = p.off, a_in[i] = p.in;
        } else {
            a_off[i] = m * (uint32_t)(g.A.ld * 4), a_in[i] = 0u;
        }
        uint32_t n = n0 + kLoadRows * i + prow;
        n = n < (uint32_t)g.N ? n : (uint32_t)g.N - 1u;
        w_off[i] = n * (uint32_t)(g.ldw * 4);
    }
    struct Group {
        u32x4 a[NA][kLoads], w[NW][kLoads];
        uint32_t skip, ky, kx;  // leading words to clear; pixels: the tap's row and column
    };
    const uint8_t *const a_base = reinterpret_cast<const uint8_t *>(g.A.base), *const w_base = reinterpret_cast<const uint8_t *>(g.W);
    auto inside = [&](const int i, const uint32_t ky, const uint32_t kx) __attribute__((always_inline)) { return (a_in[i] >> ky) & (a_in[i] >> (kx + 16u)) & 1u; };
    auto load = [&](Group &x, const SliceDigit &da, const SliceDigit &dw, const uint32_t G) __attribute__((always_inline)) {
        const Piece p = piece_of<kRows>(g, sc, (uint32_t)kPieces * G + piece0);
        x.skip = p.skip, x.ky = p.ky, x.kx = p.kx;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            uint32_t off = a_off[i] + p.off;
            // outside the image: the plane's first words, cleared below
            if constexpr (kPixels) off = inside(i, p.ky, p.kx) ? off : 0u;
            x.a[0][i] = load_piece<kRows>(a_base + da.off0 + off, sc);
            if constexpr (kA == kPair) x.a[1][i] = load_piece<kRows>(a_base + da.off1 + off, sc);
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const uint32_t off = w_off[i] + p.w_word * 4u;
            x.w[0][i] = load_piece<kRows>(w_base + dw.off0 + off, sc);
            if constexpr (kW == kPair) x.w[1][i] = load_piece<kRows>(w_base + dw.off1 + off, sc);
        }
    };
    int sum_a[kLoads] = {}, sum_w[kLoads] = {};  // row sums of this lane's pieces, current digit pair
    // registers -> LDS: fields of digit planes, plane after plane.  tail: pieces end or start within the group
    auto store = [&](Group &x, const SliceDigit &da, const SliceDigit &dw, const uint32_t G, const bool tail) __attribute__((always_inline)) {
        const uint32_t at = prow * (uint32_t)kRowBytes + ((piece0 ^ ((prow >> kSwizzle) & (kPieces - 1u))) << 4);
        // words outside the image, beyond the row's end, or brought by the piece before
        if constexpr (kPixels) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const uint32_t in = 0u - inside(i, x.ky, x.kx);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x.a[0][i][e] &= in;
                    if constexpr (kA == kPair) x.a[1][i][e] &= in;
                }
            }
        }
        if (kPixels ? (kRows == kPatches && sc.ragged) : tail) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t keep = (uint32_t)e >= x.skip ? 0xFFFFFFFFu : 0u;
#pragma unroll
                for (int i = 0; i < kLoads; ++i) {
                    x.a[0][i][e] &= keep;
                    if constexpr (kA == kPair) x.a[1][i][e] &= keep;
                }
            }
        }
        if (sc.clear_w && (kPixels || tail)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t keep = (uint32_t)e >= x.skip ? 0xFFFFFFFFu : 0u;
#pragma unroll
                for (int i = 0; i < kLoads; ++i) {
                    x.w[0][i][e] &= keep;
                    if constexpr (kW == kPair) x.w[1][i][e] &= keep;
                }
            }
        }
        if (sc.modified) {
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                apply_inversion<kA>(da.inv0, da.inv1, da.use1, x.a[0][i], x.a[NA - 1][i]);
                apply_inversion<kW>(dw.inv0, dw.inv1, dw.use1, x.w[0][i], x.w[NW - 1][i]);
            }
        }
        // (pieces beyond the last chunk are not multiplied: they count only where they are zero)
        if ((!sc.modified || (uint32_t)kPieces * G + piece0 < 2u * sc.chunks)) {
            if (sc.sum_a) {
#pragma unroll
                for (int i = 0; i < kLoads; ++i) sum_a[i] = add_sum<kA>(x.a[0][i], x.a[NA - 1][i], sum_a[i]);
            }
            if (sc.sum_w) {
#pragma unroll
                for (int i = 0; i < kLoads; ++i) sum_w[i] = add_sum<kW>(x.w[0][i], x.w[NW - 1][i], sum_w[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            u32x4 z0, z1;
            make_fields<kA>(x.a[0][i], x.a[NA - 1][i], z0, z1);
            *reinterpret_cast<u32x4 *>(lds + at + i * kLoadRows * kRowBytes) = z0;
            if constexpr (kA == kPair) *reinterpret_cast<u32x4 *>(lds + kPlaneBytes + at + i * kLoadRows * kRowBytes) = z1;
            make_fields<kW>(x.w[0][i], x.w[NW - 1][i], z0, z1);
            *reinterpret_cast<u32x4 *>(lds + NA * kPlaneBytes + at + i * kLoadRows * kRowBytes) = z0;
            if constexpr (kW == kPair) *reinterpret_cast<u32x4 *>(lds + (NA + 1) * kPlaneBytes + at + i * kLoadRows * kRowBytes) = z1;
        }
    };

    // ------------------------------------------------------------------------------------------------ products
    v16f acc[2][2];  // [n block][m block]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    // lane (r, kg) of a block reads piece 2 q + kg of row r for chunk q of the group
    const uint8_t *const pa = lds + (wm * 64u + r) * (uint32_t)kRowBytes, *const pw = lds + NA * kPlaneBytes + (wn * 64u + r) * (uint32_t)kRowBytes;
    struct Words {
        u32x4 a[NA][2], w[NW][2];
    };
    struct Operands {
        v4i a[2], w[2];
    };
    auto fetch = [&](const uint32_t q, Words &z) __attribute__((always_inline)) {
        const uint32_t piece = ((2u * q + kg) ^ ((r >> kSwizzle) & (kPieces - 1u))) << 4;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int p = 0; p < NA; ++p) z.a[p][b] = *reinterpret_cast<const u32x4 *>(pa + p * kPlaneBytes + b * 32 * kRowBytes + piece);
#pragma unroll
            for (int p = 0; p < NW; ++p) z.w[p][b] = *reinterpret_cast<const u32x4 *>(pw + p * kPlaneBytes + b * 32 * kRowBytes + piece);
        }
    };
    auto make = [&](const Words &z, const int ph, Operands &f) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; ++b) f.a[b] = make_operand<kA>(z.a[0][b], z.a[NA - 1][b], ph), f.w[b] = make_operand<kW>(z.w[0][b], z.w[NW - 1][b], ph);
    };
    auto multiply = [&](const int a_scale, const int w_scale, const uint32_t chunks) __attribute__((always_inline)) {
#pragma unroll 1
        for (uint32_t q = 0; q < chunks; ++q) {
            Words z;
            fetch(q, z);
            auto phase = [&](auto ph_tag) __attribute__((always_inline)) {
                constexpr int ph = decltype(ph_tag)::value;
                Operands f;
                make(z, ph, f);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(f.w[i]), widen(f.a[j]), acc[i][j], 4, 4, ph, w_scale, ph, a_scale);
            };
            phase(std::integral_constant<int, 0>{});
            phase(std::integral_constant<int, 1>{});
            phase(std::integral_constant<int, 2>{});
            phase(std::integral_constant<int, 3>{});
        }
    };

    const uint32_t groups = (2u * sc.chunks + kPieces - 1u) / kPieces, pairs = (uint32_t)(sc.a.count * sc.w.count);
    Group x;
    load(x, sc.a.d[0], sc.w.d[0], 0u);
    uint32_t ia = 0, iw = 0, G = 0;
    int corr_a4[kLoads] = {}, corr_w4[kLoads] = {};
    int a_scale = sc.a.d[0].scale, w_scale = sc.w.d[0].scale;
    for (uint32_t item = 0, items = pairs * groups; item < items; ++item) {
        if (item > 0) __syncthreads();  // the group before has been read
        store(x, sc.a.d[ia], sc.w.d[iw], G, 4u * kPieces * (G + 1u) > sc.row_words);
        __syncthreads();
        const uint32_t left = sc.chunks - kPieces / 2u * G;
        const bool pair_ends = G + 1u == groups;
        if (pair_ends && sc.corrected) {  // weigh the row sums of this pair
            const int shift = sc.a.d[ia].lg + sc.w.d[iw].lg;
            const int a_fac = (sc.w.d[iw].offset2 << shift) >> 1, w_fac = (sc.a.d[ia].offset2 << shift) >> 1;
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                corr_a4[i] += sum_a[i] * a_fac, corr_w4[i] += sum_w[i] * w_fac;
                sum_a[i] = 0, sum_w[i] = 0;
            }
        }
        if (++G == groups) {
            G = 0;
            if (++iw == (uint32_t)sc.w.count) iw = 0, ++ia;
        }
        const bool more = item + 1 < items;
        if (more) load(x, sc.a.d[ia], sc.w.d[iw], G);
        multiply(a_scale, w_scale, left < kPieces / 2u ? left : kPieces / 2u);
        if (more && pair_ends) a_scale = sc.a.d[ia].scale, w_scale = sc.w.d[iw].scale;
    }

    // ------------------------------------------------------------------------------------------------ epilogue
    // register v of block [i][j] is C[m][n], m = 32 j + lane mod 32, n = 32 i + 8 (v / 4) + 4 kg + v mod 4 of the wave's tile
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        if (sc.corrected) {
#pragma unroll
            for (int d = 1; d < kPieces; d <<= 1) corr_a4[i] += __shfl_xor(corr_a4[i], d, 64), corr_w4[i] += __shfl_xor(corr_w4[i], d, 64);
        }
        // (as the epilogue subtracts them: times alpha, the constant with the weight rows' part)
        if (piece0 == 0)
            corr_a[kLoadRows * i + prow] = (int)((uint32_t)corr_a4[i] * sc.alpha), corr_w[kLoadRows * i + prow] = (int)((uint32_t)corr_w4[i] * sc.alpha - sc.c0);
    }
    __syncthreads();
    float *const stage = reinterpret_cast<float *>(lds) + wave * (32 * kStagePitch);
    // (the host has checked that the sums and alpha_sum are below 2^23 in magnitude: a 24-bit product, full rate)
    const int alpha_sum = (int)sc.alpha_sum;
    auto times_alpha = [alpha_sum](const float s) __attribute__((always_inline)) { return __mul24((int)s, alpha_sum); };
    const int64_t n_wave = (int64_t)n0 + 64 * wn;
    const bool vec = (g.epi.ldc % 4 == 0) && (reinterpret_cast<uintptr_t>(g.epi.C) % 16 == 0);
    int32_t T = 0;
    bool live = false, flip = false;
    if (g.epi.T) {
        live = n_wave + lane < g.N;
        T = live ? g.epi.T[n_wave + lane] : 0;
        flip = live && g.epi.flip && g.epi.flip[n_wave + lane] != 0;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t m_blk = (int64_t)m0 + 64 * wm + 32 * j;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                *reinterpret_cast<f32x4 *>(&stage[r * kStagePitch + 32 * i + 8 * q + 4 * kg]) = v;
            }
        wave_lds_fence();
        if (!g.epi.T) {
            if (vec && n_wave + 64 <= g.N) {
                const i32x4 cw4 = *reinterpret_cast<const i32x4 *>(&corr_w[64 * wn + 4 * (lane & 15u)]);
#pragma unroll
                for (int s = 0; s < 8; ++s) {  // four rows x 256 bytes
                    const uint32_t row = 4u * s + (lane >> 4), col = 4u * (lane & 15u);
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(&stage[row * kStagePitch + col]);
                    const int ca = corr_a[64 * wm + 32 * j + row];
                    i32x4 val;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t corr = (uint32_t)ca + (uint32_t)cw4[e];
                        val[e] = (int32_t)((uint32_t)times_alpha(v[e]) - (uint32_t)corr);
                    }
                    const int64_t m = m_blk + row;
                    if (m < g.M) __builtin_nontemporal_store(val, reinterpret_cast<i32x4 *>(g.epi.C + m * g.epi.ldc + n_wave + col));
                }
            } else {
                // rows that start anywhere, or the last columns: one row per store, lanes on consecutive columns
                const int cw = corr_w[64 * wn + lane];
                const bool in = n_wave + lane < g.N;
                int32_t *dst = g.epi.C + m_blk * g.epi.ldc + n_wave + lane;
#pragma unroll 8
                for (uint32_t s = 0; s < 32; ++s) {
                    const uint32_t corr = (uint32_t)corr_a[64 * wm + 32 * j + s] + (uint32_t)cw;
                    const int32_t val = (int32_t)((uint32_t)times_alpha(stage[s * kStagePitch + lane]) - (uint32_t)corr);
                    if (in && m_blk + s < g.M) *dst = val;
                    dst += g.epi.ldc;
                }
            }
        } else {
            // a lane keeps its column; the ballot of row s is two words, kept by lanes 2 s and 2 s + 1
            const int cw = corr_w[64 * wn + lane];
            uint32_t mine = 0;
#pragma unroll 8
            for (uint32_t s = 0; s < 32; ++s) {
                const uint32_t corr = (uint32_t)corr_a[64 * wm + 32 * j + s] + (uint32_t)cw;
                const int32_t val = (int32_t)((uint32_t)times_alpha(stage[s * kStagePitch + lane]) - corr);
                const unsigned long long bits = __ballot(live && ((val >= T) != flip));
                mine = lane == 2u * s ? (uint32_t)bits : mine;
                mine = lane == 2u * s + 1u ? (uint32_t)(bits >> 32) : mine;
            }
            const int64_t m = m_blk + (lane >> 1), n = n_wave + 32 * (lane & 1u);
            if (m < g.M && n < g.N) g.epi.out_bits[m * g.epi.ldo + n / 32] = mine;
        }
        wave_lds_fence();
    }
}

typedef void (*TileFn)(const GemmArgs, const SliceArgs, const Tiles);
template <int kRows>
TileFn tile_kernel(int ka, int kw) {
    if (ka == kOne) return kw == kOne ? gemm_tile_kernel<kOne, kOne, kRows> : gemm_tile_kernel<kOne, kPair, kRows>;
    return kw == kOne ? gemm_tile_kernel<kPair, kOne, kRows> : gemm_tile_kernel<kPair, kPair, kRows>;
}

}  // namespace

int launch_gemm_tile(const GemmArgs &g, hipStream_t s) {
    SliceArgs sc;
    int ka, kw;
    if (!slice_args(g, true, sc, ka, kw)) return fail(QNN_ERR_UNSUPPORTED, "tiled FP4 kernel cannot take these arguments");
    const int64_t tiles_m = ceil_div(g.M, kTile), tiles_n = ceil_div(g.N, kTile);
    if (tiles_m * tiles_n > 0x7FFFFFFFLL) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
    const TileFn fn = !g.A.rows_are_pixels ? tile_kernel<kMatrix>(ka, kw) : (g.A.Cw < 4 ? tile_kernel<kNarrowPatches>(ka, kw) : tile_kernel<kPatches>(ka, kw));
    return QNN_LAUNCH("gemm_tile", fn, dim3((unsigned)(tiles_m * tiles_n)), dim3(kTileThreads), 0, s, g, sc, make_tiles(tiles_m, tiles_n));
}

// ---------------------------------------------------------------------------------------------------- convolution of a +-1 map
bool conv_map_supports(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N) {
    // (at least two rows and columns: a pixel is then in one of three row classes and one of three column classes)
    if (B < 1 || H < 2 || Wd < 2 || H > 32767 || Wd > 32767 || C < 1 || N < 1) return false;
    const int64_t M = B * H * Wd, Cw = words_for(C);
    if (M > 0x7FFFFF00LL || N > 0x7FFFFF00LL || 9 * ceil_div(Cw, 4) >= 32768) return false;
    if (16 * conv_class_ld(N) >= (1 << 28)) return false;  // 32-bit offsets into the class table
    if ((long double)M * Cw * 4 >= 4294967296.0L || (long double)N * 9 * Cw * 4 >= 4294967296.0L) return false;
    return 9 * Cw * 32 < 8388608 && ceil_div(M, kTile) * ceil_div(N, kTile) <= 0x7FFFFFFFLL;
}

// Tiles of 128 x 128 from which on a map is read by the kernels of whole tiles, against the sliced kernel, on the plane too or (channels that are no
// whole words, larger tiles) on the 2-bit code (App. A ConvNets, width / images of 16 x 16 to 32 x 32, us):
//   Pixels that fit LDS (qnn_gemm_image.hip), against the plane: from 40 on, where its 32 x 32 tiles end (128 / 16 of 32 x 32 52.0 -> 48.0 with the last
//   three layers sliced, 128 / 8 44.6 -> 43.0, 128 / 64 56.2 and 55.2; with the line at 64 and the 2-bit code between 96 / 32 50.7 -> 66.4); with whole
//   words, of up to 64 channels, always (32 / 1 36.8 -> 35.0, 64 / 8 38.1 -> 37.5; 96 / 1 38.5 against 40.4).
//   Against the 2-bit code: from 16 on (128 / 16 of 32 x 32 66 -> 52, 128 / 8 of 24 x 24 56 -> 51).
//   Others: from 48 on (128 / 4, 16, 64, 256 of 32 x 32 57, 74, 83, 140 with the line there, 77, 78, 84, 143 with planes alone, 58, 86, 137, 209 with
//   none, all before the kernels that hold the pixels in LDS or slice a plane).
bool conv_map_preferred(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N, bool in_lds, bool sliced) {
    const int64_t tiles = ceil_div(B * H * Wd, kTile) * ceil_div(N, kTile);
    if (!in_lds) return tiles >= 48;
    if (sliced) return tiles >= 40 || (N % 32 == 0 && C <= 64);
    return tiles >= 16;
}

int64_t conv_class_ld(int64_t N) { return ceil_div(N, kTile) * kTile; }

bool conv_map_pools(int64_t H, int64_t Wd) { return H % 2 == 0 && (Wd == 8 || Wd == 16 || Wd == 32); }

int launch_conv_map(const uint32_t *plane, int64_t B, int H, int Wd, int64_t C, const uint32_t *W, int64_t N, const uint8_t *flip_complement,
                    uint32_t *out, int64_t ldo, const int32_t *class_thr, const uint32_t *pool_and, bool pool_invert, hipStream_t s) {
    if (!conv_map_supports(B, H, Wd, C, N)) return fail(QNN_ERR_UNSUPPORTED, "convolution of a +-1 map: shape not supported");
    GemmArgs g;
    std::memset(&g, 0, sizeof(g));
    const int64_t Cw = words_for(C);
    g.A.base = plane, g.A.rows_are_pixels = 1;
    g.A.H = H, g.A.Wd = Wd, g.A.Ho = H, g.A.Wo = Wd, g.A.Cw = (int)Cw, g.A.KH = 3, g.A.KW = 3, g.A.pad = 1, g.A.stride = 1;
    g.pa.count = 1, g.pa.mode = QNN_PLANE_BIT, g.pa.coef[0] = 1;
    g.pw.count = 1, g.pw.mode = QNN_PLANE_BIT, g.pw.coef[0] = 1;
    g.W = W, g.ldw = g.Kw = 9 * Cw;
    g.epi.flip = flip_complement, g.epi.out_bits = out, g.epi.ldo = ldo;
    g.M = B * H * Wd, g.N = N, g.K = 9 * C;
    g.class_thr = class_thr, g.class_ld = conv_class_ld(N);
    g.pool_and = pool_and, g.pool_invert = pool_invert ? 0xFFFFFFFFu : 0u;
    SliceArgs sc;
    int ka, kw;
    if (!slice_args(g, true, sc, ka, kw)) return fail(QNN_ERR_UNSUPPORTED, "convolution of a +-1 map: shape not supported");
    panel::PanelArgs x;
    std::memset(&x, 0, sizeof(x));
    x.sc = sc, x.steps = (uint32_t)ceil_div(9 * (int64_t)sc.ppt, 2);
    x.a_bytes = (uint32_t)(g.M * Cw * 4), x.w_bytes = (uint32_t)(N * 9 * Cw * 4);
    int which, per;
    panel_shape(g.M, N, 8 * (int64_t)x.steps, which, per);
    const panel::Shape shape = (panel::Shape)which;
    const int64_t tiles_m = ceil_div(g.M, panel::rows_of(shape)), tiles_n = ceil_div(N, panel::columns_of(shape)), total = tiles_m * tiles_n, cus = compute_units();
    x.tiles = make_tiles(tiles_m, tiles_n);
    return QNN_LAUNCH("conv_map", panel::map_kernel(shape), dim3((unsigned)(total < per * cus ? total : per * cus)), dim3(panel::kThreads), 0, s, g, x);
}

}  // namespace qnn
