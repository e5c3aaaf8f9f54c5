// Matrix-core engine, panel-fed kernel for single-plane products on the FP4 path (the binary product of Sec. 6,
// Eq. (popc), and the hidden layers of Alg. 4).
//
//   * The workgroup brings in the operand rows it shares with loads that write straight to LDS (global_load_lds_dwordx4: no registers
//     are held while the data is on its way), 64 contiguous bytes of a row (a group of 512 elements) by four lanes: the address path
//     of a compute unit takes a cycle per line that an instruction touches, 64 for an instruction whose lanes read 64 rows, 16 here.
//     Two group buffers take turns behind one barrier per group; a group's loads are issued two steps before it is needed.
//   * A 16-byte piece c of row r sits at piece c xor (r / 4 mod 4) of its LDS row (the lanes of a load pick their global piece
//     accordingly), so that the reads (lanes = consecutive rows, same piece) use all banks; every lane reads the 16 bytes of its row
//     and k-group for the next step with one ds_read_b128 per 32-row block.
//   * Words become E2M1 operands in registers with ONE instruction per register: phase t of a step multiplies bit t of every nibble of
//     the lane's four words, and a nibble with only bit 0 / 1 / 2 set is 0.5 / 1.0 / 2.0, which the block scale of the instruction
//     (exact powers of two) turns into 1; bit 3 is the sign bit and takes a shift to bit 1.
//   * Workgroup: four waves of 64 x 32 WBN on a tile of 128 x 64 WBN (or 256 x 32 WBN), and TWO workgroups on a compute unit: one multiplies while the other
//     stores its tile (14 % of the time at 8192^3 where one workgroup of four 128 x 128 waves had the unit to itself), runs its
//     threshold epilogue or waits at its barrier.
//   * Rows (kRows): whole 64-byte groups on 16-byte boundaries; any others, starting at any word, through loads that check the
//     operand's bounds (buffer_load ... lds: what lies beyond reads as zero), the words beyond a row's end cleared in registers in its
//     last steps; or the 3 x 3 patches of a +-1 map (gemm_map_kernel below).
// Requirements (otherwise other kernels take the product): one plane per operand, operands that span less than 4 GiB each.
#pragma once
#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"
#include "qnn_gemm_slice.h"

namespace qnn {
namespace panel {

using mfma::v16f;
using mfma::v4i;

constexpr int kThreads = 256;
constexpr int WB = 2;             // blocks of 32 rows of a wave
constexpr int kRowBytes = 64;     // bytes of a row per group: two steps of two 16-byte k-groups
constexpr int kGroupWords = kRowBytes / 4;

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int t) { return t == 0 ? v.x : (t == 1 ? v.y : (t == 2 ? v.z : v.w)); }

// Thresholds of nine border classes (row class 0 = interior, 1 = first row, 2 = last row; column class likewise; 3 row + column) for the
// wave's 32 WBN filters, straight into LDS.  The table in memory is indexed by four bits (first row, last row, first column, last).
template <int WBN>
__device__ __forceinline__ void load_classes_to_lds(const GemmArgs &g, const uint32_t n_wave, float *tab, uint32_t *flip_tab) {
    const uint32_t lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float *)tab);
    const uint32_t flip_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t *)flip_tab);
    if (g.epi.flip) {
#pragma unroll
        for (uint32_t h = 0; h < WBN / 2; ++h) {
            const uint32_t n = n_wave + 64u * h + (threadIdx.x & 63u), at = n < (uint32_t)g.N ? n : (uint32_t)g.N - 1u;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ubyte %1, %2" : : "s"(flip_lds + 256u * h), "v"(at), "s"(g.epi.flip) : "memory");
        }
    }
#pragma unroll
    for (uint32_t c9 = 0; c9 < 9; ++c9) {
        const uint32_t rc = c9 / 3, cc = c9 % 3;
        const uint32_t c16 = (rc == 1 ? 1u : 0u) | (rc == 2 ? 2u : 0u) | (cc == 1 ? 4u : 0u) | (cc == 2 ? 8u : 0u);
        const int32_t *const row = g.class_thr + c16 * (uint32_t)g.class_ld + n_wave;
#pragma unroll
        for (uint32_t h = 0; h < WBN / 2; ++h)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(lds + (c9 * 32u * WBN + 64u * h) * 4u), "v"((64u * h + (threadIdx.x & 63u)) * 4u), "s"(row) : "memory");
    }
}

// Epilogue of a map: register v of block [bi][bj] belongs to pixel m = m_wave + 32 bj + lane mod 32 and filter 32 bi + 8 (v / 4) + 4 kg + v
// mod 4 of the wave's; the sign bit of threshold - S is appended with a funnel shift per element, and every lane ends up with its pixel's
// (m_wave + lane) words of 32 filters.  The 2 x 2 max-pooling that may follow (OR of the four bits where the threshold does not flip,
// AND where it does) is two exchanges of those words (maps 8, 16 or 32 pixels wide and of even height: the wave's 64 pixels are 8, 4 or 2
// rows, the first of them even).
template <int WBN>
__device__ __forceinline__ void map_finish(const GemmArgs &g, const slice::SliceArgs &sc, v16f (&acc)[WBN][WB], int32_t (&ra)[WB], const float *tab, const uint32_t *flip_tab,
                                           const uint32_t m_wave, const uint32_t n_wave) {
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));
    const uint32_t r = lane & 31u, kg = lane >> 5;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the thresholds landed long ago, before a barrier)
    const float *at[WB];
    float sum[WB];
#pragma unroll
    for (int j = 0; j < WB; ++j) {
        uint32_t rem, px;
        (void)slice::quotient(m_wave + 32u * j + r, (uint32_t)(g.A.H * g.A.Wd), sc.inv_hw, rem);
        const uint32_t py = slice::quotient(rem, (uint32_t)g.A.Wd, sc.inv_w, px);
        const uint32_t c9 = 3u * (py == 0u ? 1u : (py + 1u == (uint32_t)g.A.H ? 2u : 0u)) + (px == 0u ? 1u : (px + 1u == (uint32_t)g.A.Wd ? 2u : 0u));
        at[j] = tab + c9 * (32u * WBN) + 4u * kg;
        sum[j] = (float)mfma::sum_halves(ra[j]);
    }
    uint32_t word[WBN], use_and[WBN];
#pragma unroll
    for (int i = 0; i < WBN; ++i) use_and[i] = g.pool_and && n_wave + 32u * i < (uint32_t)g.N ? g.pool_and[n_wave / 32u + i] ^ g.pool_invert : 0u;
#pragma unroll
    for (int i = 0; i < WBN; ++i) {
        const uint32_t n = n_wave + 32u * i;
        const uint32_t live = (uint32_t)__ballot(n + r < (uint32_t)g.N), flips = (uint32_t)__ballot(flip_tab[32 * i + r] != 0u);
        uint32_t both[WB];
#pragma unroll
        for (int j = 0; j < WB; ++j) {
            uint32_t bits = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 t4 = *reinterpret_cast<const float4 *>(at[j] + 32 * i + 8 * q);
                const float thr[4] = {t4.x, t4.y, t4.z, t4.w};
                uint32_t nib = 0;
#pragma unroll
                for (int e = 3; e >= 0; --e)  // S = 2 acc - sum > threshold  <=>  threshold + sum - 2 acc < 0
                    nib = __builtin_amdgcn_alignbit(nib, __float_as_uint(__builtin_fmaf(-2.0f, acc[i][j][4 * q + e], thr[e] + sum[j])), 31);
                bits |= nib << (8 * q);
            }
            both[j] = mfma::or_halves(bits << (4u * kg));
        }
        word[i] = ((kg ? both[1] : both[0]) ^ flips) & live;
        __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t *dst;
    bool mine;
    if (!g.pool_and) {
        mine = m_wave + lane < (uint32_t)g.M;
        dst = g.epi.out_bits + (int64_t)(m_wave + lane) * g.epi.ldo + n_wave / 32u;
    } else {
        const int below = g.A.Wd;  // lanes between a pixel and the one below it
#pragma unroll
        for (int i = 0; i < WBN; ++i) {
            const uint32_t mask = use_and[i];
            auto merge = [mask](const uint32_t a, const uint32_t b) { return ((a | b) & ~mask) | (a & b & mask); };
            const uint32_t v = merge(word[i], (uint32_t)__shfl_xor((int)word[i], below, 64));
            word[i] = merge(v, (uint32_t)__shfl_xor((int)v, 1, 64));
        }
        uint32_t px;
        const uint32_t row0 = slice::quotient(m_wave, (uint32_t)g.A.Wd, sc.inv_w, px);  // row of the first pixel, over all images (even heights)
        const uint32_t sy = lane / (uint32_t)g.A.Wd, sx = lane - sy * (uint32_t)g.A.Wd;
        mine = m_wave + lane < (uint32_t)g.M && ((sy | sx) & 1u) == 0u;
        dst = g.epi.out_bits + ((int64_t)((row0 + sy) / 2u) * (g.A.Wd / 2) + sx / 2u) * g.epi.ldo + n_wave / 32u;
    }
    if (!mine) return;
    if (WBN == 4 && g.epi.ldo % 4 == 0 && reinterpret_cast<uintptr_t>(g.epi.out_bits) % 16 == 0 && n_wave + 128u <= (uint32_t)g.N) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(word[0], word[1], word[WBN - 2], word[WBN - 1]);
    } else {
#pragma unroll
        for (int i = 0; i < WBN; ++i)
            if (n_wave + 32u * i < (uint32_t)g.N) dst[i] = word[i];
    }
}

enum Rows { kWholeRows = 0, kAnyRows = 1, kMapRows = 2 };
struct PanelArgs {
    Tiles tiles;
    uint32_t steps;             // of 256 elements
    uint32_t a_bytes, w_bytes;  // kAnyRows, kMapRows: sizes of the operands
    slice::SliceArgs sc;        // kMapRows: how the patches are found
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// LDS of a workgroup: two group buffers, then per wave either the weight rows' terms and the thresholds and flip flags, or the weight rows'
// terms and a 32 x 32 staging block, through which a block of int32 sums is turned from the accumulator layout (a lane = one row) into
// whole 128-byte lines per row; kMapRows: the thresholds of nine border classes.
template <Rows kRows, bool kSign, int WM, int WBN>
constexpr uint32_t kLdsBytes = 2 * (64 * WM + 32 * WBN * (4 / WM)) * kRowBytes + 4 * (kRows == kMapRows ? 10 * 32 * WBN * 4 : (kSign ? 3 * 512 : 512 + 4096));

// kSign: threshold epilogue (Alg. 4: a^b = Sign(BatchNorm(a))) instead of int32 sums.
// WM: waves along m, 2 or 4; WBN: 32-column blocks per wave along n, 2 or 4.
// kMapRows (3 x 3 "same" convolutions of +-1 maps, pad 1, stride 1, threshold output): the left operand is the map's plane "value is -1"
// (0 outside the image).  With a = 1 - 2 p inside the image, conv = sum_{taps inside} sum_c w - 2 S, S = sum_k p w = 2 sum_k p b - sum_k p,
// so a pixel's bit is (S > class_thr[class][n]) xor flip[n], class = which of the image's borders the pixel lies on (see prepare_block).
template <Rows kRows, bool kSign, int WM, int WBN>
__device__ __forceinline__ void panel_product(const GemmArgs &g, const MfmaConst &mc, const PanelArgs &x, uint8_t *const lds) {
    static_assert(kRows != kMapRows || kSign, "maps are thresholded");
    constexpr int WN = 4 / WM, BM = 64 * WM, WTN = 32 * WBN, BN = WN * WTN;  // rows of the tile, columns of a wave / of the tile
    constexpr uint32_t kPanelBytes = BM * kRowBytes, kGroupBytes = kPanelBytes + BN * kRowBytes;
    const uint32_t ngroups = (x.steps + 1u) / 2u;

    const uint32_t lane = threadIdx.x & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave / WN, wn = wave % WN;
    const uint32_t total_tiles = x.tiles.total;
    auto opaque = [](uint32_t x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    // this wave's tables / staging block
    uint8_t *const tail = lds + 2 * kGroupBytes + wave * (kRows == kMapRows ? 10u * WTN * 4u : (kSign ? 3u * 512u : 512u + 4096u));
    float *const class_tab = reinterpret_cast<float *>(tail);
    uint32_t *const rw_tab = reinterpret_cast<uint32_t *>(tail);
    int32_t *const thr_tab = reinterpret_cast<int32_t *>(tail + 512), *const stage_w = thr_tab;
    uint32_t *const flip_tab = reinterpret_cast<uint32_t *>(tail + (kRows == kMapRows ? 9u * WTN * 4u : 1024u));
    if constexpr (kSign) {  // flip flags default to "none" (complete long before the first epilogue reads them)
        flip_tab[lane] = 0u;
        if (kRows != kMapRows || WBN == 4) flip_tab[lane + 64] = 0u;
    }
    const uint32_t lds_base = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds);

    // ------------------------------------------------------------------------------------------------ producer
    // A load instruction of a wave covers 16 consecutive rows x 64 bytes and fills 1 KiB of LDS: lane i lands in slot i mod 4 of row
    // i / 4, so it fetches piece (i mod 4) xor (row / 4 mod 4).  Load i of a panel takes rows 64 i + 16 wave .. + 15.  The cursor (a
    // tile, group p_G) runs two groups ahead of the multiplication; what depends on the tile only (the byte offsets of the rows this
    // lane loads, with its piece) is worked out when it enters a tile.
    // This workgroup's tiles: vb0, vb0 + gridDim.x, ... (n_mine of them).
    constexpr int kLoadsA = BM / 64, kLoadsW = BN / 64, kLoads = kLoadsA + kLoadsW;
    const uint32_t vb0 = blockIdx.x, n_mine = (total_tiles - vb0 + gridDim.x - 1u) / gridDim.x;
    uint32_t p_G = 0, p_item = 0;
    uint32_t off[kLoads], in[kRows == kMapRows ? kLoadsA : 1];  // kMapRows: of the patch, and which of its taps lie inside (see patch_of)
    auto p_locate = [&](const uint32_t vb) __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(vb, x.tiles, tm, tn);
        const uint32_t ln = opaque(lane), row = 16u * wave + (ln >> 2), piece = ((ln & 3u) ^ (ln >> 4)) << 4;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const bool is_a = i < kLoadsA;
            const uint32_t last = (uint32_t)((is_a ? g.M : g.N) - 1);
            uint32_t at = (is_a ? tm * (uint32_t)BM + 64u * i : tn * (uint32_t)BN + 64u * (i - kLoadsA)) + row;
            at = at > last ? last : at;
            if (kRows == kMapRows && is_a) {
                const slice::Patch p = slice::patch_of(g, x.sc, at);
                off[i] = p.off, in[i % kLoadsA] = p.in;
            } else {
                off[i] = at * ((uint32_t)(is_a ? g.A.ld : g.ldw) * 4u) + (kRows == kMapRows ? 0u : piece);
            }
        }
    };
    auto p_advance = [&]() __attribute__((always_inline)) {
        if (++p_G == ngroups) {
            asm volatile("" ::: "memory");  // keeps the branch a branch
            p_G = 0;
            ++p_item;
            // (after the last tile the loads are repeated and never used)
            p_locate(p_item < n_mine ? vb0 + p_item * gridDim.x : vb0);
        }
    };
    auto resource = [](const void *base, const uint32_t bytes) __attribute__((always_inline)) {
        const uint64_t p = reinterpret_cast<uint64_t>(base);
        return u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xFFFFu, bytes, 0x00027000u};
    };
    const u32x4 a_rsrc = resource(g.A.base, x.a_bytes), w_rsrc = resource(g.W, x.w_bytes);
    // kMapRows: this lane's piece of the group at the cursor
    struct Tap {
        uint32_t off, w_off, ky, kx;
    } tap = {0u, 0u, 0u, 0u};
    auto p_tap = [&]() __attribute__((always_inline)) {
        if constexpr (kRows == kMapRows) {
            const uint32_t ln = opaque(lane), piece = 4u * p_G + ((ln & 3u) ^ (ln >> 4));
            uint32_t t = __umulhi(piece, x.sc.magic_ppt);
            if (x.sc.ppt == 1u) t = piece;
            const uint32_t word = 4u * (piece - t * x.sc.ppt);
            tap.ky = (t * 11u) >> 5, tap.kx = t - 3u * tap.ky;  // t / 3 for t < 32
            tap.w_off = t < 9u ? (t * x.sc.row_words + word) * 4u : 0xFFFFFFF0u;
            if (t >= 9u) tap.ky = 15u;  // a tap row that no patch has
            tap.off = ((tap.ky * (uint32_t)g.A.Wd + tap.kx) * x.sc.row_words + word) * 4u;
        }
    };
    auto load = [&](const int i, const uint32_t buf) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + buf + (uint32_t)i * 4096u + wave * 1024u;
        const bool is_a = i < kLoadsA;
        if constexpr (kRows == kWholeRows) {
            const uint8_t *const base = reinterpret_cast<const uint8_t *>(is_a ? g.A.base : g.W) + p_G * (uint32_t)kRowBytes;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off[i]), "s"(base) : "memory");
        } else {
            uint32_t voff;
            if constexpr (kRows == kAnyRows) {
                voff = off[i] + p_G * (uint32_t)kRowBytes;
            } else {
                const bool inside = ((in[i % kLoadsA] >> tap.ky) & (in[i % kLoadsA] >> (tap.kx + 16u)) & 1u) != 0u;
                voff = is_a ? (inside ? off[i] + tap.off : 0xFFFFFFF0u) : (tap.w_off == 0xFFFFFFF0u ? tap.w_off : off[i] + tap.w_off);
            }
            if (is_a)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(dst), "v"(voff), "s"(a_rsrc) : "memory");
            else
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(dst), "v"(voff), "s"(w_rsrc) : "memory");
        }
    };
    // the next group has landed and this wave's LDS reads have returned
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // (the second group may still be on its way)
    auto first_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kLoads) : "memory"); };

    p_locate(vb0);
    p_tap();
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(i, 0u);
    p_advance();
    p_tap();
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(i, kGroupBytes);
    first_barrier();
    uint32_t rd = 0u;  // byte offset of the group buffer being consumed

    // ------------------------------------------------------------------------------------------------ consumer
    struct Step {
        uint4 A[WB], W[WBN];
    };
    // lane (r, kg) of a block reads piece 2 q + kg of row r at step q of a group
    auto fetch = [&](const uint32_t q, const uint32_t buf, Step &d) __attribute__((always_inline)) {
        const uint32_t at = buf + r * (uint32_t)kRowBytes + (((2u * q + kg) ^ ((r >> 2) & 3u)) << 4);
        const uint8_t *const pa = lds + (at + wm * (uint32_t)(32 * WB * kRowBytes)), *const pw = lds + (at + kPanelBytes + wn * (uint32_t)(WTN * kRowBytes));
#pragma unroll
        for (int b = 0; b < WB; ++b) d.A[b] = *reinterpret_cast<const uint4 *>(pa + b * (32 * kRowBytes));
#pragma unroll
        for (int b = 0; b < WBN; ++b) d.W[b] = *reinterpret_cast<const uint4 *>(pw + b * (32 * kRowBytes));
    };
    v16f acc[WBN][WB];  // [n block][m block]
    int32_t ra[WB], rw[WBN];
    auto operand = [](const uint4 &c, const int t) __attribute__((always_inline)) {
        v4i f;
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = (int)(t == 3 ? (word_of(c, j) >> 2) & 0x22222222u : word_of(c, j) & (0x11111111u << t));
        // An E2M1 operand is four registers; the upper four of the builtin's type stay undefined
        return __builtin_shufflevector(f, f, 0, 1, 2, 3, -1, -1, -1, -1);
    };
    // block scales of the four phases as E8M0 bytes (2^(e - 127)): 2, 1, 1/2, 1
    const int scales = 0x7F7E7F80;
    // Phase t: 32 of a step's 128 elements per lane, and the counts of one word of every row (each made opaque after its addition:
    // left alone, the compiler keeps the counts of a whole loop trip in registers of their own)
    auto phase = [&](auto t_tag, const Step &c, auto between) __attribute__((always_inline)) {
        constexpr int t = decltype(t_tag)::value;
        mfma::v8i a[WB];
#pragma unroll
        for (int j = 0; j < WB; ++j) a[j] = operand(c.A[j], t);
#pragma unroll
        for (int i = 0; i < WBN; ++i) {
            const auto w = operand(c.W[i], t);
#pragma unroll
            for (int jj = 0; jj < WB; ++jj) {
                const int j = i & 1 ? WB - 1 - jj : jj;  // (one operand stays from one instruction to the next)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, a[j], acc[i][j], 4, 4, t, scales, t, scales);
            }
            if constexpr (kRows != kMapRows) {
                rw[i] += (int32_t)__builtin_popcount(word_of(c.W[i], t));
                asm("" : "+v"(rw[i]));
            }
            between(i);
        }
#pragma unroll
        for (int j = 0; j < WB; ++j) {
            ra[j] += (int32_t)__builtin_popcount(word_of(c.A[j], t));
            asm("" : "+v"(ra[j]));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    std::integral_constant<int, 0> p0;
    std::integral_constant<int, 1> p1;
    std::integral_constant<int, 2> p2;
    std::integral_constant<int, 3> p3;
    auto nothing = [](int) __attribute__((always_inline)) {};
    // Words of step q of group G that are not the rows' own: beyond a row's end (kAnyRows: in both operands, whose bits are counted), or
    // beyond a pixel's channels (kMapRows: in the map alone)
    auto clear_surplus = [&](const uint32_t G, const uint32_t q, Step &c) __attribute__((always_inline)) {
        if constexpr (kRows == kAnyRows) {
            if (8u * (2u * G + q) + 8u > (uint32_t)g.Kw) {
                const uint32_t first = 8u * (2u * G + q) + 4u * kg, have = (uint32_t)g.Kw > first ? (uint32_t)g.Kw - first : 0u;
                const uint32_t k0 = have > 0u ? ~0u : 0u, k1 = have > 1u ? ~0u : 0u, k2 = have > 2u ? ~0u : 0u, k3 = have > 3u ? ~0u : 0u;
#pragma unroll
                for (int b = 0; b < WB; ++b) c.A[b].x &= k0, c.A[b].y &= k1, c.A[b].z &= k2, c.A[b].w &= k3;
#pragma unroll
                for (int b = 0; b < WBN; ++b) c.W[b].x &= k0, c.W[b].y &= k1, c.W[b].z &= k2, c.W[b].w &= k3;
            }
        } else if constexpr (kRows == kMapRows) {
            if (x.sc.ragged) {
                const uint32_t piece = 2u * (2u * G + q) + kg;
                const uint32_t t = x.sc.ppt == 1u ? piece : __umulhi(piece, x.sc.magic_ppt), word = 4u * (piece - t * x.sc.ppt), have = x.sc.row_words - word;
                const uint32_t k1 = have > 1u ? ~0u : 0u, k2 = have > 2u ? ~0u : 0u, k3 = have > 3u ? ~0u : 0u;
#pragma unroll
                for (int b = 0; b < WB; ++b) c.A[b].y &= k1, c.A[b].z &= k2, c.A[b].w &= k3;
            }
        }
    };

    Step cur, nxt;
    fetch(0, rd, cur);
    uint32_t vb = vb0;
    for (uint32_t done = 0; done < n_mine; ++done, vb += gridDim.x) {
        uint32_t tile_m, tile_n;
        tile_of_block(vb, x.tiles, tile_m, tile_n);
        const int64_t m_wave = (int64_t)tile_m * BM + wm * (32 * WB), n_wave = (int64_t)tile_n * BN + wn * WTN;
#pragma unroll
        for (int j = 0; j < WB; ++j) ra[j] = 0;
#pragma unroll
        for (int i = 0; i < WBN; ++i) {
            rw[i] = 0;
#pragma unroll
            for (int j = 0; j < WB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        }
        // thresholds and flip flags of this tile on their way to the wave's LDS tables (free since the previous tile's epilogue)
        if constexpr (kSign && kRows != kMapRows) load_thresholds_to_lds<WBN>(g, n_wave, thr_tab, flip_tab);
        if constexpr (kRows == kMapRows) load_classes_to_lds<WBN>(g, (uint32_t)n_wave, class_tab, flip_tab);
        for (uint32_t G = 0; G < ngroups; ++G) {
            const uint32_t other = kGroupBytes - rd;
            p_advance();
            p_tap();
            fetch(1, rd, nxt);
            clear_surplus(G, 0u, cur);
            __builtin_amdgcn_sched_barrier(0);
            phase(p0, cur, nothing);
            phase(p1, cur, nothing);
            phase(p2, cur, nothing);
            phase(p3, cur, nothing);
            barrier();  // every wave holds the second step's words: the buffer is free
            fetch(0, other, cur);
            if (kRows != kWholeRows && 2u * G + 1u == x.steps) {  // (nothing in the group's second step)
#pragma unroll
                for (int i = 0; i < kLoads; ++i) load(i, rd);
                rd = other;
                break;
            }
            clear_surplus(G, 1u, nxt);
            __builtin_amdgcn_sched_barrier(0);
            phase(p0, nxt, [&](const int i) __attribute__((always_inline)) {
                constexpr int kEach = (kLoads + WBN - 1) / WBN;
#pragma unroll
                for (int p = 0; p < kEach; ++p)
                    if (kEach * i + p < kLoads) load(kEach * i + p, rd);
            });
            phase(p1, nxt, nothing);
            phase(p2, nxt, nothing);
            phase(p3, nxt, nothing);
            rd = other;
        }
        // The sums are pinned here: otherwise the compiler moves matrix-core instructions down into the epilogue's blocks
#pragma unroll
        for (int i = 0; i < WBN; ++i)
#pragma unroll
            for (int j = 0; j < WB; ++j) asm volatile("" : "+v"(acc[i][j]));
        if constexpr (kRows == kMapRows)
            map_finish<WBN>(g, x.sc, acc, ra, class_tab, flip_tab, (uint32_t)m_wave, (uint32_t)n_wave);
        else
            wave_finish<kSign, WBN, kLoads, kBothTerms>(g, mc, acc, ra, rw, rw_tab, thr_tab, flip_tab, stage_w, m_wave, n_wave);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads beyond the last tile)
}

template <bool kSign, int WM, int WBN, int kRows>
__global__ __launch_bounds__(kThreads, 2) void gemm_panel_kernel(const GemmArgs g, const MfmaConst mc, const PanelArgs x) {
    static_assert(kLdsBytes<(Rows)kRows, kSign, WM, WBN> <= 80 * 1024, "two workgroups on a compute unit");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kLdsBytes<(Rows)kRows, kSign, WM, WBN>];
    panel_product<(Rows)kRows, kSign, WM, WBN>(g, mc, x, lds);
}

// The same for a +-1 map
template <int WM, int WBN>
__global__ __launch_bounds__(kThreads, 2) void gemm_map_kernel(const GemmArgs g, const PanelArgs x) {
    static_assert(kLdsBytes<kMapRows, true, WM, WBN> <= 80 * 1024, "two workgroups on a compute unit");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kLdsBytes<kMapRows, true, WM, WBN>];
    const MfmaConst none = {};
    panel_product<kMapRows, true, WM, WBN>(g, none, x, lds);
}

// Tiles and how many workgroups of them share a compute unit
enum Shape { k128x256 = 0, k128x128 = 1, k256x128 = 2 };
constexpr int64_t rows_of(Shape t) { return t == k256x128 ? 256 : 128; }
constexpr int64_t columns_of(Shape t) { return t == k128x256 ? 256 : 128; }

typedef void (*KernelFn)(const GemmArgs, const MfmaConst, const PanelArgs);
typedef void (*MapFn)(const GemmArgs, const PanelArgs);
// whole: rows of whole 64-byte groups on 16-byte boundaries
KernelFn find_kernel(bool sign, Shape shape, bool whole);
MapFn map_kernel(Shape shape);
typedef void (*WideFn)(const GemmArgs, const MfmaConst, uint32_t, uint32_t, uint32_t);
WideFn wide_kernel();  // int32 sums, 256 x 256 tiles, rows of whole 128-byte groups (qnn_gemm_panel_wide_kernel.h)
constexpr int kWideGroupWords = 32;

}  // namespace panel
}  // namespace qnn
