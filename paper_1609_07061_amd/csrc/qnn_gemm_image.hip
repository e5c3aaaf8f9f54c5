// Matrix-core kernels for 3 x 3 "same" convolutions (pad 1, stride 1) with +-1 filters: the +-1 maps of a ConvNet (threshold output,
// max-pooling) and images of bit planes (int32 sums or thresholds).
//
// Bound before: a tile's patches came to LDS tap by tap and every wave made its operands of them, nine times per pixel: 5.5 and more vector
// instructions per matrix-core instruction, where 4 go by unnoticed (a SIMD issues for 15 cycles per 32 x 32 x 64 FP4 instruction and 4 per
// vector instruction, and the former holds the matrix core for 32).  Here
//   * a workgroup brings the pixels that its tile's patches are made of to LDS once, as E2M1 operands: a word of 32 channels is 16 bytes, the
//     nibble 4 j + t of the word's bits in nibble j of dword t.  +-1 maps are +-1, two planes of neighbouring powers a digit 0 .. 3, and what
//     lies outside the image 0, so that nothing has to be corrected for the border: the sums are the convolution's own.  Rows of pixels have a
//     zero pixel in front (which ends the row before, too), images a zero row: pixel (y, x) of image b is LDS pixel
//     (b (H + 1) + y + 1) (W + 1) + x + 1 less the tile's first, a tap a constant distance.
//   * an operand of the left side is one 16-byte LDS read, at the lane's pixel plus the word's distance from a table.  An odd number of 16-byte
//     pieces per pixel spreads the reads of neighbouring pixels over all banks.
//   * filters stay bits (groups of 512 through three LDS buffers, loads that write LDS directly, as in qnn_gemm_panel_kernel.h): a word
//     becomes +-1 operands with seven instructions, which 32 PB pixels of the wave share.
//   * max-pooling: the pixels are numbered window by window, so that the four of a window are neighbouring lanes.
//   * thresholds: the sums start from 1/2 - T, so that a finished sum's sign is its bit.
// Workgroup: 2 x 2 waves of 32 PB pixels x 32 NB filters, several on a compute unit: one stages its pixels while others multiply.
// What is left (App. A's layers on 256 images): the matrix cores' time, 0.9 of it in the loop, and 2 to 3 us at the start and end of every round of
// tiles that nothing covers, since all of them start at once.  Five layers 98 -> 75 us (under the profiler), the whole forward pass 111 -> 88.4; one image of 32 x 32
// and 32 filters 54 -> 36.
#include <cstring>

#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"
#include "qnn_gemm_slice.h"

namespace qnn {
namespace image {

namespace {

using mfma::v16f;
using mfma::v4i;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // a 16-byte load at any word

constexpr int kThreads = 256;
constexpr uint32_t kGroupWords = 16, kRowBytes = 4 * kGroupWords;  // of a filter per group

struct ImageArgs {
    const uint32_t *planes;   // the map's plane "value is -1", or the first bit plane
    uint64_t plane_stride;    // words
    int count;                // bit planes
    uint32_t H, W, Cw, C;     // C: channels (maps)
    uint32_t images;
    uint32_t inv_w1, inv_h1, inv_pieces, inv_words;  // floor(2^32 / .) of W + 1, H + 1, pieces and words of a pixel (2^32 - 1 for 1)
    uint32_t inv_row, inv_all;                       // ... of the output's (pooled: windows') row and image
    uint32_t row, all;                               // pixels (pooled: windows) of a row and an image of the output
    uint32_t pitch;           // bytes of an LDS pixel
    uint32_t tile_bytes;      // LDS pixels of the largest tile
    uint32_t tiles_m, tiles_n, inv_tiles_n;
    uint32_t plane_bytes;     // size of a plane
    uint32_t flip_bytes;      // of the flip flags (0: none)
    uint32_t w_bytes;         // size of the filters
    uint32_t invert;          // thresholds: all ones if the bit is (sum >= T) xor flip, 0 if it is that inverted
    const uint32_t *pool_and; // 2 x 2 max-pooling: packed flags of the filters whose bits are AND-ed, inverted with pool_invert (null: none)
    uint32_t pool_invert;
    uint32_t *ones;           // maps: receives the output's "inside the image" plane, laid out like the output (null: not wanted)
};

template <int PB, int NB>
constexpr uint32_t kFixedBytes = 3 * 64 * NB * kRowBytes + 64 * NB * 4;  // filters, what the sums start from

template <int PB, int NB, bool kMap, bool kSign>
__device__ __forceinline__ void product(const GemmArgs &g, const ImageArgs &x, uint8_t *const lds) {
    constexpr uint32_t BM = 64 * PB, BN = 64 * NB, kGroup = BN * kRowBytes;
    static_assert(PB == 2 || PB == 4, "words are stored for pairs of blocks");
    const uint32_t t = threadIdx.x, lane = t & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 1, wn = wave & 1u;
    // consecutive tiles on one XCD (workgroups congruent mod 8), those of the same pixels together
    const uint32_t xcd = blockIdx.x & 7u, in_all = gridDim.x >> 3, left_over = gridDim.x & 7u;
    uint32_t tn;
    const uint32_t tm = quotient(xcd * in_all + (xcd < left_over ? xcd : left_over) + (blockIdx.x >> 3), x.tiles_n, x.inv_tiles_n, tn);
    const uint32_t m0 = tm * BM, n0 = tn * BN, M = (uint32_t)g.M, N = (uint32_t)g.N;
    const bool pooled = kSign && x.pool_and != nullptr;

    // LDS: pixels, filters (three groups), what the sums start from, distances
    uint8_t *const filters = lds + x.tile_bytes;
    float *const start_tab = reinterpret_cast<float *>(filters + 3 * kGroup);
    int32_t *const dist_tab = reinterpret_cast<int32_t *>(start_tab + BN);
    const uint32_t lds_filters = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds) + x.tile_bytes;

    // ------------------------------------------------------------------------------------------------ pixels
    // padded row (see above) and column of output pixel m
    auto locate = [&](uint32_t m, uint32_t &row, uint32_t &col) __attribute__((always_inline)) {
        m = m < M ? m : M - 1u;  // (pixels beyond the last repeat it and are not stored)
        const uint32_t at = pooled ? m >> 2 : m;
        uint32_t rem, xx;
        const uint32_t b = quotient(at, x.all, x.inv_all, rem);
        uint32_t y = quotient(rem, x.row, x.inv_row, xx);
        if (pooled) y = 2u * y + ((m >> 1) & 1u), xx = 2u * xx + (m & 1u);
        row = b * (x.H + 1u) + y + 1u, col = xx + 1u;
    };
    uint32_t row0, row1, col;
    locate(m0, row0, col);
    locate(m0 + BM - 1u, row1, col);
    row0 -= 1u;
    const uint32_t pixels = (row1 + 2u - row0) * (x.W + 1u) + 1u, pieces = (x.Cw + 3u) / 4u;
    // Pixels to LDS, four words of a pixel per thread and turn: asked for, and put there
    constexpr int kAhead = kMap ? 4 : 2;  // pieces whose loads are on their way together
    struct Piece {
        u32x4 v0, v1;
        uint8_t *dst;
        uint32_t sign, plus_one, first;  // first: channel
    };
    const uint32_t count = pixels * pieces;
    auto load4 = [&](const uint32_t *base, const uint32_t at) __attribute__((always_inline)) {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(base), 0, (int)x.plane_bytes, 0x00027000);
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0));
    };
    auto ask = [&](const uint32_t d, const uint32_t i, Piece &p) __attribute__((always_inline)) {
        const bool second = !kMap && 2u * d + 1u < (uint32_t)x.count;
        uint32_t piece, c, yy;
        const uint32_t pixel = quotient(i, pieces, x.inv_pieces, piece), pr = quotient(pixel, x.W + 1u, x.inv_w1, c);
        const uint32_t b = quotient(row0 + pr, x.H + 1u, x.inv_h1, yy);
        const bool inside = yy != 0u && c != 0u && b < x.images;
        // (outside the image: beyond the plane, which reads as zeros; a ragged pixel's last piece reads the next pixel's words along)
        const uint32_t src = inside && i < count ? (((b * x.H + yy - 1u) * x.W + c - 1u) * x.Cw + 4u * piece) * 4u : 0xFFFFFFF0u;
        const uint32_t *const p0 = x.planes + (kMap ? 0u : 2u * d * x.plane_stride);
        p.v0 = load4(p0, src);
        if constexpr (!kMap) p.v1 = load4(p0 + (second ? x.plane_stride : 0u), second ? src : 0xFFFFFFF0u);
        p.dst = lds + pixel * x.pitch + 64u * piece;
        p.sign = inside ? 0x88888888u : 0u, p.plus_one = inside ? 0x22222222u : 0u;
        p.first = 128u * piece;
    };
    const bool whole = x.C % 128u == 0u;  // pixels of whole pieces
    auto put = [&](const Piece &p) __attribute__((always_inline)) {
        auto expand = [&](const int e) __attribute__((always_inline)) {
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (kMap)
                    o[q] = ((p.v0[e] << (3 - q)) & p.sign) | p.plus_one;
                else
                    o[q] = ((p.v0[e] >> q) & 0x11111111u) | (((p.v1[e] >> q) & 0x11111111u) << 1);
            }
            return o;
        };
        if (whole) {
#pragma unroll
            for (int e = 0; e < 4; ++e) *reinterpret_cast<u32x4 *>(p.dst + 16 * e) = expand(e);
        } else {
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                if (p.first + 32u * e >= 32u * x.Cw) continue;
                u32x4 o = expand((int)e);
                const uint32_t left = x.C - (p.first + 32u * e);  // channels from here on
                if (left < 32u) {
                    const uint32_t live = (1u << left) - 1u;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t there = (live >> q) & 0x11111111u;
                        o[q] &= (there << 4) - there;  // (the nibbles that exist; a carry out of the last is lost)
                    }
                }
                *reinterpret_cast<u32x4 *>(p.dst + 16u * e) = o;
            }
        }
    };
    Piece piece[kAhead];
    auto ask_all = [&](const uint32_t d, const uint32_t first) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k)
            if (first - t + k * kThreads < count) ask(d, first + k * kThreads, piece[k]);  // (a branch of the whole workgroup)
    };
    auto put_all = [&](const uint32_t first) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k)
            if (first + k * kThreads < count) put(piece[k]);
    };
    // ------------------------------------------------------------------------------------------------ filters
    // A load of a wave covers 16 rows x 64 bytes; piece c of row r sits at piece c xor (r / 4 mod 4).
    const uint32_t Kw = (uint32_t)g.Kw, full = Kw / kGroupWords, rest = Kw % kGroupWords, groups = full + (rest ? 1u : 0u);
    const uint64_t w_base = reinterpret_cast<uint64_t>(g.W);
    const u32x4 w_rsrc = {(uint32_t)w_base, (uint32_t)(w_base >> 32) & 0xFFFFu, x.w_bytes, 0x00027000u};
    uint32_t w_off[BN / 64];
#pragma unroll
    for (uint32_t i = 0; i < BN / 64; ++i) {
        uint32_t n = n0 + 64u * i + 16u * wave + (lane >> 2);
        n = n < N ? n : N - 1u;
        w_off[i] = n * (Kw * 4u) + (((lane & 3u) ^ (lane >> 4)) << 4);
    }
    auto load_group = [&](const uint32_t G, const uint32_t buf) __attribute__((always_inline)) {
#pragma unroll
        for (uint32_t i = 0; i < BN / 64; ++i) {
            const uint32_t dst = lds_filters + buf + i * 4096u + wave * 1024u, voff = w_off[i] + G * kRowBytes;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(dst), "v"(voff), "s"(w_rsrc) : "memory");
        }
    };
    // three groups take turns, so that a load has two groups' time (the digits start over; behind the last the loads are repeated, never used)
    uint32_t p_G = 0;
    auto load_next = [&](const uint32_t buf) __attribute__((always_inline)) {
        load_group(p_G, buf);
        p_G = p_G + 1u == groups ? 0u : p_G + 1u;
    };
    load_next(0u);
    if constexpr (kMap) ask_all(0u, t);
    const uint32_t digits = kMap ? 1u : (uint32_t)(x.count + 1) / 2u;

    // thresholds, flip flags and the pooling's flags, asked for before the tables are made
    int32_t threshold = 0;
    uint32_t flip[NB] = {};
    uint32_t pool_mask[NB] = {};
    if constexpr (kSign) {
        threshold = g.epi.T[n0 + t % BN < N ? n0 + t % BN : N - 1u];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const uint32_t n = n0 + (wn * NB + i) * 32u;
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(g.epi.flip), 0, (int)x.flip_bytes, 0x00027000);
            flip[i] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rsrc, (int)(n + r), 0, 0);
            const auto flags = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(x.pool_and), 0, pooled ? (int)((N + 31u) / 32u * 4u) : 0, 0x00027000);
            uint32_t at = n / 32u * 4u;
            asm volatile("" : "+v"(at));  // (as a value of the whole wave it would be waited for here)
            pool_mask[i] = __builtin_amdgcn_raw_buffer_load_b32(flags, (int)at, 0, 0);
        }
    }

    // ------------------------------------------------------------------------------------------------ tables
    for (uint32_t kw = t; kw < (groups + 1u) * kGroupWords; kw += kThreads) {
        uint32_t word, kx;
        const uint32_t tap = quotient(kw, x.Cw, x.inv_words, word), ky = (tap * 11u) >> 5;  // tap / 3 for tap < 32
        kx = tap - 3u * ky;
        dist_tab[kw] = kw < Kw ? (((int32_t)ky - 1) * (int32_t)(x.W + 1u) + (int32_t)kx - 1) * (int32_t)x.pitch + 16 * (int32_t)word : 0;
    }

    uint32_t base[PB];  // this lane's pixels
#pragma unroll
    for (int j = 0; j < PB; ++j) {
        uint32_t row;
        locate(m0 + (wm * PB + j) * 32u + r, row, col);
        base[j] = ((row - row0) * (x.W + 1u) + col) * x.pitch;
    }

    // ------------------------------------------------------------------------------------------------ products
    v16f acc[NB][PB];  // [filters][pixels]
    // what the wave's LDS reads have returned, and the next group has landed
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const uint8_t *const filter_row = filters + (wn * 32u * NB + r) * kRowBytes;
    const uint32_t turn = (r >> 2) & 3u;
    uint32_t plus = 0x22222222u, minus = 0xAAAAAAAAu;  // (registers: with literals in their place the compiler takes an instruction more)
    asm volatile("" : "+v"(plus), "+v"(minus));
    // the products of a word of every filter with the pixels' operands; kFirst: the sums start from `start`
    v16f start[NB];
    auto multiply = [&](auto first_tag, const uint32_t (&w)[NB], const v4i (&a)[PB], const int scale) __attribute__((always_inline)) {
        constexpr bool kFirst = decltype(first_tag)::value;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            v4i f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t bits = w[i] << (3 - q);
                f[q] = (int)((bits & plus) | (~bits & minus));
            }
            const mfma::v8i f8 = __builtin_shufflevector(f, f, 0, 1, 2, 3, -1, -1, -1, -1);
#pragma unroll
            for (int j = 0; j < PB; ++j) {
                const mfma::v8i a8 = __builtin_shufflevector(a[j], a[j], 0, 1, 2, 3, -1, -1, -1, -1);
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f8, a8, kFirst ? start[i] : acc[i][j], 4, 4, 0, 0x7F7F7F7F, 0, scale);
            }
        }
    };
    auto read_pixels = [&](const int32_t dist, v4i (&a)[PB]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < PB; ++j) a[j] = *reinterpret_cast<const v4i *>(lds + (base[j] + (uint32_t)dist));
    };
    struct Step {  // eight words of every filter: lane half kg has words 4 kg .. + 3 of them
        uint4 w[NB];
        int4 dist;
    };
    auto fetch = [&](const uint32_t G, const uint32_t q, const uint32_t at, Step &s) __attribute__((always_inline)) {
        const uint8_t *const p = filter_row + (at + (((2u * q + kg) ^ turn) << 4));
#pragma unroll
        for (int i = 0; i < NB; ++i) s.w[i] = *reinterpret_cast<const uint4 *>(p + i * 32 * kRowBytes);
        s.dist = *reinterpret_cast<const int4 *>(dist_tab + G * kGroupWords + 8u * q + 4u * kg);
    };
    // A step's four products; the pixels' operands are read two words ahead of their use (those of the first two are there)
    v4i a0[PB], a1[PB], a2[PB];
    auto step = [&](auto first_tag, const Step &s, const int4 &next, const int scale) __attribute__((always_inline)) {
        uint32_t w[NB];
        read_pixels(s.dist.z, a2);
#pragma unroll
        for (int i = 0; i < NB; ++i) w[i] = s.w[i].x;
        multiply(first_tag, w, a0, scale);
        __builtin_amdgcn_sched_barrier(0);
        read_pixels(s.dist.w, a0);
#pragma unroll
        for (int i = 0; i < NB; ++i) w[i] = s.w[i].y;
        multiply(std::false_type{}, w, a1, scale);
        __builtin_amdgcn_sched_barrier(0);
        v4i b0[PB];
        read_pixels(next.x, b0);
#pragma unroll
        for (int i = 0; i < NB; ++i) w[i] = s.w[i].z;
        multiply(std::false_type{}, w, a2, scale);
        __builtin_amdgcn_sched_barrier(0);
        read_pixels(next.y, a1);
#pragma unroll
        for (int i = 0; i < NB; ++i) w[i] = s.w[i].w;
        multiply(std::false_type{}, w, a0, scale);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < PB; ++j) a0[j] = b0[j];
    };

    uint32_t buf = 0;  // the group buffer being multiplied
    auto after = [&](const uint32_t at) __attribute__((always_inline)) { return at == 2u * kGroup ? 0u : at + kGroup; };
    // the next group has landed (the one behind it may be on its way), and this wave's LDS reads have returned
    auto barrier_ahead = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(BN / 64) : "memory"); };
    for (uint32_t d = 0; d < digits; ++d) {
        if (d > 0) barrier();  // the digit before has been multiplied
        if constexpr (kMap) put_all(t);
        for (uint32_t i = kMap ? t + kAhead * kThreads : t; i < count; i += kAhead * kThreads) {
            ask_all(d, i);
            put_all(i);
        }
        if constexpr (kSign) {
            // (sums are below 2^21 in magnitude: clamping thresholds there changes no comparison, and halves stay exact)
            if (d == 0 && t < BN) start_tab[t] = 0.5f - (float)(threshold < -(1 << 21) ? -(1 << 21) : (threshold > (1 << 21) ? (1 << 21) : threshold));
        }
        if (d == 0) {
            load_next(kGroup);
            load_next(2u * kGroup);
        }
        // The first group has landed, the two behind it may be on their way.  (Every wave waits for its own part of it: one without a pixel to stage has
        // waited for no load so far.)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(2 * BN / 64) : "memory");
        if (d == 0) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if constexpr (kSign) v = *reinterpret_cast<const float4 *>(&start_tab[(wn * NB + i) * 32 + 8 * q + 4 * kg]);
                    start[i][4 * q] = v.x, start[i][4 * q + 1] = v.y, start[i][4 * q + 2] = v.z, start[i][4 * q + 3] = v.w;
                }
            if (!kMap || full == 0u) {  // (a map's first products start from these registers)
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j < PB; ++j) acc[i][j] = start[i];
            }
        }
        // a digit's nibble n is n / 2
        const int scale = kMap ? 0x7F7F7F7F : (int)(0x80808080u + d * 0x02020202u);
        if (full) {
            Step s0, s1;
            fetch(0u, 0u, buf, s0);
            read_pixels(s0.dist.x, a0);
            read_pixels(s0.dist.y, a1);
            uint32_t G = 0;
            auto group = [&](auto first_tag) __attribute__((always_inline)) {
                fetch(G, 1u, buf, s1);
                step(first_tag, s0, s1.dist, scale);
                barrier_ahead();  // every wave holds the second step's words: the buffer is free
                load_next(buf);
                buf = after(buf);
                fetch(++G, 0u, buf, s0);  // (behind the last group: not used)
                step(std::false_type{}, s1, s0.dist, scale);
            };
            if constexpr (kMap) group(std::true_type{});
            while (G < full) group(std::false_type{});
        }
        if (rest) {
            // the words that are left, one per lane half at a time; a word that does not exist meets the zero pixel in front
            for (uint32_t u = 0; 2u * u < rest; ++u) {
                const uint32_t word = 2u * u + kg;
                const int32_t dist = dist_tab[full * kGroupWords + word];
                uint32_t w[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) w[i] = *reinterpret_cast<const uint32_t *>(filter_row + (buf + (((word >> 2) ^ turn) << 4) + 4u * (word & 3u)) + i * 32 * kRowBytes);
#pragma unroll
                for (int j = 0; j < PB; ++j) a0[j] = *reinterpret_cast<const v4i *>(lds + (word < rest ? base[j] + (uint32_t)dist : 0u));
                multiply(std::false_type{}, w, a0, scale);
            }
            if (d + 1u < digits) {
                barrier();
                load_next(buf);
            }
            buf = after(buf);
        }
    }

    // ------------------------------------------------------------------------------------------------ epilogue
    // The sums are pinned here: otherwise the compiler moves matrix-core instructions down into the epilogue
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < PB; ++j) asm volatile("" : "+v"(acc[i][j]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads behind the last group)
    const uint32_t m_wave = m0 + wm * 32u * PB, n_wave = n0 + wn * 32u * NB;
    if constexpr (!kSign) {
        barrier();  // the pixels have been read: their room takes the blocks on their way out
        mfma::MfmaConst mc = {};
        mc.alpha = (uint32_t)g.pa.coef[0], mc.alpha_shift = g.pa.coef[0] == 1 ? 0 : -1;
        int32_t ra[PB] = {}, rw[NB] = {};
        panel::wave_finish<false, NB, 0, panel::kNoTerms>(g, mc, acc, ra, rw, nullptr, nullptr, nullptr, reinterpret_cast<int32_t *>(lds) + wave * 1024, m_wave, n_wave);
    } else {
        // register 4 q + e of block [i][j]: filter 32 i + 8 q + 4 kg + e, pixel 32 j + r of the wave's; a finished sum is negative where the
        // convolution is below the threshold
        uint32_t flips[NB], live[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const uint32_t n = n_wave + 32u * i;
            live[i] = n >= N ? 0u : (N - n >= 32u ? 0xFFFFFFFFu : (1u << (N - n)) - 1u);
            flips[i] = (uint32_t)__ballot(flip[i] != 0u) ^ x.invert;
        }
        // a block's words of 32 filters, in both lane halves
        auto words = [&](const int j, uint32_t (&word)[NB]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t nib = 0;
#pragma unroll
                    for (int e = 3; e >= 0; --e) nib = __builtin_amdgcn_alignbit(nib, __float_as_uint(acc[i][j][4 * q + e]), 31);
                    bits |= nib << (8 * q);
                }
                uint32_t v = (mfma::or_halves(bits << (4u * kg)) ^ flips[i]) & live[i];
                if (pooled) {
                    // OR of the window's four bits where the threshold does not flip, AND where it does
                    const uint32_t mask = pool_mask[i] ^ x.pool_invert;
                    auto merge = [mask](const uint32_t a, const uint32_t b) { return ((a | b) & ~mask) | (a & b & mask); };
                    v = merge(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));  // lane xor 1
                    v = merge(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));  // lane xor 2
                }
                word[i] = v;
            }
        };
        // lane half kg stores the blocks kg, 2 + kg
#pragma unroll
        for (int jj = 0; jj < PB; jj += 2) {
            uint32_t even[NB], odd[NB];
            words(jj, even);
            words(jj + 1, odd);
            const uint32_t m = m_wave + 32u * (jj + kg) + r;
            if (m >= M || (pooled && (m & 3u) != 0u)) continue;
            uint32_t *const dst = g.epi.out_bits + (int64_t)(pooled ? m >> 2 : m) * g.epi.ldo + n_wave / 32u;
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (n_wave + 32u * i < N) dst[i] = kg ? odd[i] : even[i];
            if (kMap && x.ones) {
                uint32_t *const inside = x.ones + (dst - g.epi.out_bits);
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (n_wave + 32u * i < N) inside[i] = live[i];
            }
        }
    }
}

constexpr int waves_per_simd(int PB) { return PB == 2 ? 3 : 2; }

// +-1 maps, 2 x 2 waves of 32 PB x 64
template <int PB>
__global__ __launch_bounds__(kThreads, waves_per_simd(PB)) void gemm_map_image_kernel(const GemmArgs g, const ImageArgs x) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    product<PB, 2, true, true>(g, x, lds);
}
// images of bit planes
template <int PB, int NB, bool kSign>
__global__ __launch_bounds__(kThreads, waves_per_simd(PB)) void gemm_image_kernel(const GemmArgs g, const ImageArgs x) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    product<PB, NB, false, kSign>(g, x, lds);
}

// LDS pixels of the largest tile of `tile` pixels (pooled: of whole windows): rows that the tile's pixels lie on, zero rows between images,
// a row above and one below.
int64_t tile_pixels(int64_t H, int64_t W, bool pooled, int64_t tile) {
    const int64_t row = pooled ? W / 2 : W, all = row * (pooled ? H / 2 : H), n = pooled ? tile / 4 : tile;
    const int64_t rows = n % row == 0 ? n / row : (n - 2) / row + 2, images = all % n == 0 ? 1 : (n % all == 0 ? n / all : (n - 2) / all + 2);
    // (a pooled image of odd height has a row that no window covers)
    return ((pooled ? 2 : 1) * rows + (images - 1) * (pooled && H % 2 ? 2 : 1) + 2) * (W + 1) + 1;
}

constexpr int64_t kMostLds = 80 * 1024;  // two workgroups on a compute unit

// Everything but the operands; false if the kernels cannot take the shape.
bool plan(int64_t B, int64_t H, int64_t W, int64_t C, int64_t N, bool pooled, int PB, int64_t &M, ImageArgs &x, int64_t &lds_bytes) {
    std::memset(&x, 0, sizeof(x));
    if (B < 1 || H < 1 || W < 1 || C < 1 || N < 1 || H > 32767 || W > 32767) return false;
    const int64_t Cw = words_for(C), row = pooled ? W / 2 : W, all = row * (pooled ? H / 2 : H), tile = 64 * PB;
    if (all < 1 || B * H * W > 0x7FFFFF00LL || B * (H + 1) > 0x7FFFFF00LL || N > 0x7FFFFF00LL || (long double)N * 9 * Cw * 4 >= 4294967000.0L) return false;
    if ((long double)B * H * W * Cw * 4 >= 4294967000.0L) return false;  // (offsets beyond stand for what lies outside)
    M = B * all * (pooled ? 4 : 1);
    const int64_t pitch = (Cw | 1) * 16, pixels = tile_pixels(H, W, pooled, tile), groups = ceil_div(9 * Cw, kGroupWords);
    lds_bytes = pixels * pitch + (PB == 2 ? kFixedBytes<2, 2> : kFixedBytes<4, 2>) + (groups + 1) * kGroupWords * 4;
    if (pixels * pitch < 4 * 4096) lds_bytes += 4 * 4096 - pixels * pitch;  // (the blocks of int32 sums)
    if (lds_bytes > kMostLds || ceil_div(M, tile) * ceil_div(N, 128) > 0x7FFFFFFFLL) return false;
    x.H = (uint32_t)H, x.W = (uint32_t)W, x.Cw = (uint32_t)Cw, x.C = (uint32_t)C, x.images = (uint32_t)B;
    x.inv_w1 = inverse_of(W + 1), x.inv_h1 = inverse_of(H + 1), x.inv_pieces = inverse_of(ceil_div(Cw, 4)), x.inv_words = inverse_of(Cw);
    x.inv_tiles_n = inverse_of(ceil_div(N, 128)), x.plane_bytes = (uint32_t)(B * H * W * Cw * 4);
    x.row = (uint32_t)row, x.all = (uint32_t)all, x.inv_row = inverse_of(row), x.inv_all = inverse_of(all);
    x.pitch = (uint32_t)pitch, x.tile_bytes = (uint32_t)(pixels * pitch < 4 * 4096 ? 4 * 4096 : pixels * pitch);
    x.tiles_m = (uint32_t)ceil_div(M, tile), x.tiles_n = (uint32_t)ceil_div(N, 128), x.w_bytes = (uint32_t)(N * 9 * Cw * 4);
    return true;
}

}  // namespace

// Blocks of 32 pixels of a wave, 4 or 2, by the time of the tiles' rounds: a tile's own time (tables, pixels, epilogue) and the matrix
// instructions of all that share a compute unit (us; of App. A's layers on 256 images, 4 / 2: 32 x 32, 128 -> 128 channels, 1024 / 2048 tiles,
// 19.7 / 22.7; 16 x 16, 128 -> 256, 512 / 1024, 11.1 / 12.8, 256 -> 256 18.3 / 19.6; 8 x 8, 256 -> 512, 256 / 512, 13.0 / 11.7).  0: the pixels
// do not fit.
struct Plan {
    int PB;
    ImageArgs x;
    int64_t M, lds_bytes;
};
static int blocks(int64_t B, int64_t H, int64_t W, int64_t C, int64_t N, bool pooled, int digits, Plan &best) {
    best.PB = 0;
    double least = 0.0;
    const int64_t cus = compute_units();
    for (int PB = 2; PB <= 4; PB += 2) {
        Plan p;
        p.PB = PB;
        if (!plan(B, H, W, C, N, pooled, PB, p.M, p.x, p.lds_bytes)) continue;
        const int64_t tiles = (int64_t)p.x.tiles_m * p.x.tiles_n, per = PB == 2 && 3 * p.lds_bytes <= 160 * 1024 ? 3 : 2, rest = tiles % (per * cus);
        const double own = PB == 2 ? 3.0 : 3.6, products = 0.0134 * PB * 9.0 * (double)words_for(C) * digits;
        const double us = (double)(tiles / (per * cus)) * (own + (double)per * products) + (rest ? own + (double)ceil_div(rest, cus) * products : 0.0);
        if (best.PB == 0 || us < least) best = p, least = us;
    }
    return best.PB;
}

bool map_supports(int64_t B, int64_t H, int64_t W, int64_t C, int64_t N, bool pooled) {
    Plan p;
    return 9 * C < (1 << 21) && blocks(B, H, W, C, N, pooled, 1, p) != 0;
}

int launch_map(const uint32_t *plane, int64_t B, int H, int W, int64_t C, const uint32_t *filters, int64_t N, const int32_t *T, const uint8_t *flip_complement,
               uint32_t *out, uint32_t *ones, int64_t ldo, const uint32_t *pool_and, bool pool_invert, hipStream_t s) {
    Plan p;
    ImageArgs &x = p.x;
    if (blocks(B, H, W, C, N, pool_and != nullptr, 1, p) == 0) return fail(QNN_ERR_UNSUPPORTED, "convolution of a +-1 map: shape not supported");
    GemmArgs g;
    std::memset(&g, 0, sizeof(g));
    g.M = p.M, g.N = N, g.K = 9 * C, g.Kw = 9 * words_for(C), g.W = filters;
    g.epi.T = T, g.epi.flip = flip_complement, g.epi.out_bits = out, g.epi.ldo = ldo;
    x.planes = plane, x.count = 1, x.flip_bytes = flip_complement ? (uint32_t)N : 0u, x.pool_and = pool_and, x.pool_invert = pool_invert ? 0xFFFFFFFFu : 0u, x.ones = ones;
    return QNN_LAUNCH("conv_map", (p.PB == 4 ? gemm_map_image_kernel<4> : gemm_map_image_kernel<2>), dim3(x.tiles_m * x.tiles_n), dim3(kThreads), (unsigned)p.lds_bytes, s, g, x);
}

// A convolution's arguments: images of bit planes 1, 2, 4, ... times a factor (0: something else), +-1 filters.
static int32_t factor(const GemmArgs &g) {
    const LeftAddr &a = g.A;
    if (!a.rows_are_pixels || a.KH != 3 || a.KW != 3 || a.pad != 1 || a.stride != 1) return 0;
    if (g.pa.mode != QNN_PLANE_BIT || g.pw.mode != QNN_PLANE_SIGN || g.pw.count != 1 || g.ldw != g.Kw) return 0;
    for (int p = 1; p < g.pa.count; ++p)
        if ((int64_t)g.pa.coef[p] != (int64_t)g.pa.coef[0] << p) return 0;
    const int64_t f = (int64_t)g.pa.coef[0] * g.pw.coef[0];
    return f > -0x7FFFFFFF && f < 0x7FFFFFFF ? (int32_t)f : 0;
}

bool conv_supports(const GemmArgs &g) {
    const int64_t f = factor(g), most = 9 * 32 * (int64_t)g.A.Cw * ((1 << g.pa.count) - 1);
    // thresholds start the sums in halves: below 2^21; int32 sums are whole numbers below 2^24
    if (f == 0 || (g.epi.T && f != 1) || most >= (g.epi.T ? 1 << 21 : 1 << 24)) return false;
    const int64_t B = g.M / ((int64_t)g.A.H * g.A.Wd);
    Plan p;
    return blocks(B, g.A.H, g.A.Wd, 32 * (int64_t)g.A.Cw, g.N, false, (g.pa.count + 1) / 2, p) != 0;
}

// From 128 tiles of 128 x 128 on (1090 convolutions of 1 to 1000 images of 6 x 6 to 112 x 112, 3 to 384 channels, 8 to 701 filters, 1, 2 and 4 bits: 0.93
// to 7 times as fast there as on the tiled kernel, us there / here: 37 x 28 x 28, 64 -> 192, 4 bits 23.3 / 11.7; 202 x 15 x 15, 238 -> 128, 2 bits 22.1 / 13.8; 256
// x 13 x 13, 384 -> 256, 2 bits 30.2 / 23.8; below on the sliced kernel 0.3 to 1.1), but not
//   * where half of a tile's 128 filters are missing and the patches are long (255 x 21 x 21, 207 -> 64, 1 bit 17.5 / 21.2; 54 x 28 x 28, 128 -> 64, 2 bits
//     11.1 / 9.1);
//   * for int32 sums where three quarters are missing (35 x 32 x 32, 128 -> 32, 2 bits 6.5 / 9.5, 32 -> 8, 1 bit 5.9 / 7.3), nor on one bit where the 64 are not
//     full (66 x 56 x 56, 64 -> 48 23.7 / 28.1) or the patch has more than two words a tap (24 x 24, 128 -> 64 7.9 / 8.7, 64 -> 64 8.5 / 7.5), nor on two where they are
//     not full and it has more than three (131 x 14 x 14, 128 -> 48 7.6 / 8.8);
//   * for one or two bits and sums beyond the cache in rows of no whole lines that three tiles and more share: a line's parts reach memory apart there
//     (79 x 64 x 64, 9 -> 331, 1 bit, 428 MB 154 / 209, 332 filters 157 / 167; 300 x 28 x 28, 311 MB 117 / 90).
bool conv_preferred(const GemmArgs &g) {
    if (ceil_div(g.M, 128) * ceil_div(g.N, 128) < 128) return false;
    const int64_t words = (int64_t)g.A.Cw * ((g.pa.count + 1) / 2);
    const bool sums = g.epi.T == nullptr;
    if (g.N <= 64 && words > 4) return false;
    if (sums && g.N <= 32) return false;
    if (sums && g.N <= 64 && g.pa.count == 1 && (g.N < 64 || words > 2)) return false;
    if (sums && g.N < 64 && g.pa.count == 2 && words > 3) return false;
    if (sums && g.N > 256 && g.N % 32 != 0 && g.pa.count <= 2 && (g.N % 4 != 0 || words == 1) && 4.0 * (double)g.M * (double)g.N > 384e6) return false;
    return conv_supports(g);
}

int launch_conv(const GemmArgs &given, hipStream_t s) {
    Plan p;
    ImageArgs &x = p.x;
    GemmArgs g = given;
    const int64_t B = g.M / ((int64_t)g.A.H * g.A.Wd), C = 32 * (int64_t)g.A.Cw;  // (what lies beyond the channels is zero bits)
    if (blocks(B, g.A.H, g.A.Wd, C, g.N, false, (g.pa.count + 1) / 2, p) == 0) return fail(QNN_ERR_UNSUPPORTED, "convolution: shape not supported");
    x.planes = g.A.base, x.plane_stride = (uint64_t)g.A.plane_stride, x.count = g.pa.count;
    x.flip_bytes = g.epi.flip ? (uint32_t)g.N : 0u, x.invert = 0xFFFFFFFFu;
    g.pa.coef[0] = factor(given);
    auto kernel = g.epi.T ? (p.PB == 4 ? gemm_image_kernel<4, 2, true> : gemm_image_kernel<2, 2, true>)
                          : (p.PB == 4 ? gemm_image_kernel<4, 2, false> : gemm_image_kernel<2, 2, false>);
    return QNN_LAUNCH("conv_image", kernel, dim3(x.tiles_m * x.tiles_n), dim3(kThreads), (unsigned)p.lds_bytes, s, g, x);
}

}  // namespace image
}  // namespace qnn
