// Operand description shared by the two FP4 kernels for products of any size and layout (qnn_gemm_slice.hip,
// qnn_gemm_tile.hip): digits of an operand, and how a 256-element chunk of a digit becomes E2M1 operands.
#pragma once
#include <cstring>
#include <utility>

#include "qnn_internal.h"

namespace qnn {
namespace slice {

using qnn::quotient;

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // a 16-byte load at any word

constexpr int kMaxDigits = QNN_MAX_PLANES;

// How an operand's planes enter the multiplication.
enum SliceKind {
    kPm1 = 0,   // every digit is one +-1 plane, multiplied as +-1
    kPair = 1,  // every digit is one or two 0/1 planes, multiplied as a number 0 .. 3
    kOne = 2,   // every digit is one plane, multiplied as 0 / 1 (a +-1 plane too: 2 b - 1 = 2 (b - 1/2))
    kMap = 3    // one plane "value is -1" of a +-1 map whose channels fill whole words, 0 outside the image (sliced kernel, left operand)
};
// The digit's value is 2^lg (u - offset2 / 2), u = the number made of its planes' bits (as inverted).
struct SliceDigit {
    uint32_t off0, off1;  // byte offsets of the planes from the operand's base (off1 = off0 where there is no second one)
    uint32_t inv0, inv1;  // all ones if the plane's bits are inverted
    uint32_t use1;        // kPair: all ones if the second plane exists, else 0
    int offset2;
    int lg;
    int scale;            // E8M0 bytes of the instruction's block scale for the four phases of a chunk
};
struct SliceOperand {
    int count;
    SliceDigit d[kMaxDigits];
};
struct SliceArgs {
    SliceOperand a, w;
    uint32_t chunks;       // 256-element chunks of a row (pixels: of KH KW taps padded to whole pieces each)
    uint32_t row_words;    // words of a row (pixels: of a tap) = Kw (Cw)
    uint32_t ppt, taps;    // pixels: 16-byte pieces per tap, taps
    uint32_t magic_ppt, magic_kw;  // ceil(2^32 / .)
    uint32_t inv_hw, inv_w;        // pixels: floor(2^32 / .) of the output map's pixels and width (2^32 - 1 for 1)
    // C = alpha_sum S - alpha (row corrections) + c0; S counts a +-1 plane that is multiplied as 0 / 1 with its bit, not with twice its
    // bit, and alpha_sum is alpha times two for every operand of such planes
    uint32_t alpha, alpha_sum, c0;
    int corrected;       // some digit has an offset: row sums are taken
    int modified;        // some digit has an inverted or an absent plane
    int sum_a, sum_w;    // the left / right operand's row sums are wanted
    int ragged;          // the rows (pixels: the taps) are not made of whole pieces
    int clear_w;         // +-1 activation planes: where activation words are cleared the weight words have to be cleared too
};

// Fields for the operands of a digit, from its planes' words: a single plane as it lies; a pair of planes as two-bit fields
// (b1 b0), those of the even bits in z0, of the odd bits in z1.
//   A 0/1 plane with a negative coefficient enters inverted, -b = (1 - b) - 1, so every field is a number 0 .. 3 and its operand
//   one mask away; with x = ua - oa, y = uw - ow the product sum is  sum ua uw - ow sum ua - oa sum uw + K oa ow,  row sums that
//   cost a few population counts per 128 elements instead of four to five instructions per eight elements for signs.
template <int kKind>
__device__ __forceinline__ void make_fields(const u32x4 &w0, const u32x4 &w1, u32x4 &z0, u32x4 &z1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (kKind == kPair) {
            const uint32_t f0 = (w0[i] & 0x55555555u) | ((w1[i] << 1) & 0xAAAAAAAAu);
            const uint32_t f1 = ((w0[i] >> 1) & 0x55555555u) | (w1[i] & 0xAAAAAAAAu);
            z0[i] = f0, z1[i] = f1;
        } else {
            z0[i] = w0[i];
        }
    }
}
// The planes' bits as the digit counts them: inverted where the coefficient is negative, the second plane absent or not.
template <int kKind>
__device__ __forceinline__ void apply_inversion(const uint32_t inv0, const uint32_t inv1, const uint32_t use1, u32x4 &w0, u32x4 &w1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w0[i] ^= inv0;
        if constexpr (kKind == kPair) w1[i] = (w1[i] ^ inv1) & use1;
    }
}
// sum + the sum of u over the 128 elements
template <int kKind>
__device__ __forceinline__ int add_sum(const u32x4 &w0, const u32x4 &w1, int sum) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (kKind == kPair)
            sum += __builtin_popcount(w0[i]) + 2 * __builtin_popcount(w1[i]);
        else if constexpr (kKind == kOne)
            sum += __builtin_popcount(w0[i]);
        else
            sum += 2 * __builtin_popcount(w0[i]) - 32;
    }
    return sum;
}
// E2M1 operand of phase ph: bit ph of every nibble of the words.
template <int kKind>
__device__ __forceinline__ v4i make_operand(const u32x4 &z0, const u32x4 &z1, const int ph) {
    v4i f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (kKind == kMap) {
            f[i] = (int)(((z0[i] << (3 - ph)) & 0x88888888u) | z1[i]);  // (z1: 1.0 in every nibble, or nothing)
        } else if constexpr (kKind == kPair) {
            const uint32_t z = (ph & 1) ? z1[i] : z0[i];
            f[i] = (int)(((ph & 2) ? (z >> 2) : z) & 0x33333333u);
        } else if constexpr (kKind == kOne) {
            // bit 0, 1 or 2 of a nibble alone is 0.5, 1 or 2 (the block scale of the phase makes it 1); bit 3 is the sign bit
            // and goes to bit 1 first
            f[i] = (int)(ph == 3 ? (z0[i] >> 2) & 0x22222222u : z0[i] & (0x11111111u << ph));
        } else {
            const uint32_t s = z0[i] << (3 - ph);
            f[i] = (int)((~s & 0x88888888u) | 0x22222222u);
        }
    }
    return f;
}
__device__ __forceinline__ v8i widen(const v4i &x) { return __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1); }

// How the rows of the left operand are found (LeftAddr): a matrix, the patches of an image, or those of an image whose pixels have
// fewer than four words.
enum SliceRows { kMatrix = 0, kPatches = 1, kNarrowPatches = 2 };

// 16 bytes of a row; narrow pixels word by word, the rest zero
template <int kRows>
__device__ __forceinline__ u32x4 load_piece(const uint8_t *p, const SliceArgs &sc) {
    if constexpr (kRows == kNarrowPatches) {
        const uint32_t *w = reinterpret_cast<const uint32_t *>(p);
        u32x4 v = {w[0], 0u, 0u, 0u};
        if (sc.row_words > 1u) v.y = w[1];
        if (sc.row_words > 2u) v.z = w[2];
        return v;
    } else {
        return *reinterpret_cast<const u32x4_any *>(p);
    }
}

// The patch of output pixel m: byte offset of its first tap's pixel (modulo 2^32: the tap may lie outside the image) and which
// of its tap rows (bits 0 .. 15) and tap columns (bits 16 .. 31) lie inside.
struct Patch {
    uint32_t off, in;
};
// quads: the rows come in fours of the pixels that 2 x 2 pooling makes one, and Ho, Wo and the quotients are the pooled map's.
__device__ __forceinline__ Patch patch_of(const GemmArgs &g, const SliceArgs &sc, const uint32_t m, const bool quads = false) {
    const uint32_t per = (uint32_t)(g.A.Ho * g.A.Wo);
    uint32_t rem, xo;
    const uint32_t img = quotient(quads ? m >> 2 : m, per, sc.inv_hw, rem);
    uint32_t yo = quotient(rem, (uint32_t)g.A.Wo, sc.inv_w, xo);
    if (quads) yo = 2u * yo + ((m >> 1) & 1u), xo = 2u * xo + (m & 1u);
    const int y = (int)yo * g.A.stride - g.A.pad, x = (int)xo * g.A.stride - g.A.pad;
    auto inside = [](const int first, const int taps, const int size) {  // taps t with 0 <= first + t < size
        const int lo = first < 0 ? (-first < 16 ? -first : 16) : 0, end = size - first;
        const int hi = end < taps ? (end > 0 ? end : 0) : taps;
        return hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
    };
    Patch p;
    p.off = (img * (uint32_t)(g.A.H * g.A.Wd) + (uint32_t)(y * g.A.Wd + x)) * sc.row_words * 4u;
    p.in = inside(y, g.A.KH, g.A.H) | (inside(x, g.A.KW, g.A.Wd) << 16);
    return p;
}
// A lane's piece of the rows: first word within the row (pixels: the tap) and within the weight row, leading words to clear;
// pixels: the tap's row and column, the byte offset from the first tap's pixel.
struct Piece {
    uint32_t word, w_word, skip, ky, kx, off;
};
template <int kRows>
__device__ __forceinline__ Piece piece_of(const GemmArgs &g, const SliceArgs &sc, const uint32_t piece) {
    Piece p;
    if constexpr (kRows == kMatrix) {
        p.word = p.w_word = 4u * piece < sc.row_words - 4u ? 4u * piece : sc.row_words - 4u;
        p.skip = 4u * piece - p.word;
        p.ky = p.kx = 0u;
        p.off = p.word * 4u;
    } else {
        uint32_t tap = __umulhi(piece, sc.magic_ppt);
        if (sc.ppt == 1u) tap = piece;  // (ceil(2^32 / 1) does not fit)
        const uint32_t sub = piece - tap * sc.ppt;
        p.word = sc.ppt == 1u || 4u * sub < sc.row_words - 4u ? 4u * sub : sc.row_words - 4u;
        p.skip = 4u * sub - p.word;
        p.ky = 0u;
        if (tap >= sc.taps) tap = 0u, p.skip = 4u, p.ky = 15u;  // beyond the patch: a tap row that no patch has
        uint32_t q = __umulhi(tap, sc.magic_kw);
        if (g.A.KW == 1) q = tap;
        p.kx = tap - q * (uint32_t)g.A.KW;
        p.off = ((q * (uint32_t)g.A.Wd + p.kx) * sc.row_words + p.word) * 4u;
        p.ky |= q;
        p.w_word = tap * sc.row_words + p.word;
    }
    return p;
}

// The kernels' arguments for a product and the kinds of its operands; false if they cannot take it.  bits: +-1 planes as kOne (with
// corrections from row sums) instead of kPm1, and a lone 0/1 plane on the right as kOne instead of kPair (on the left it always is).
bool slice_args(const GemmArgs &g, bool bits, SliceArgs &sc, int &kind_a, int &kind_w);

}  // namespace slice
}  // namespace qnn
