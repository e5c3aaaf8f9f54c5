// The backward step's products on FP6 gradients (see qnn_gemm_mixed_kernel.h): the kernels that write the operands' images, the choice
// of tiles and the launches.
#include <cstring>

#include "qnn_bitsplit.h"
#include "qnn_gemm_mixed_kernel.h"

namespace qnn {
namespace mixed {

namespace {

typedef uint32_t v6u __attribute__((ext_vector_type(6)));

// Packed bits transposed into a bits image: the image's rows are the matrix's columns, its k the matrix's rows.
struct BitsJob {
    const uint32_t *in;
    int64_t rows, cols, ld;  // (ld in words)
    uint8_t *out;
    uint32_t out_rows, groups, blocks;  // rows of an image's group; groups of 256; workgroups of this job
};
// A thread takes 32 rows x one word, rows in the order in which their bits lie in an image's word, so that the transposition of its
// 32 x 32 block gives finished words.  A workgroup takes 256 rows x 32 words: four threads have the four words of an image row.
__device__ __forceinline__ void transpose_to_image(const BitsJob &job, const uint32_t block) {
    const uint32_t G = block % job.groups;
    const uint32_t j = block / job.groups * 32u + (threadIdx.x >> 3), h = (threadIdx.x >> 2) & 1u, i = threadIdx.x & 3u;
    if ((int64_t)j >= (job.cols + 31) / 32) return;
    const int64_t r0 = 256 * (int64_t)G + 128 * h + 8 * i;
    uint32_t x[32];
#pragma unroll
    for (int p = 0; p < 32; ++p) {  // bit t of nibble n: row 32 t + n
        const int64_t row = r0 + 32 * (p & 3) + (p >> 2);
        x[p] = row < job.rows ? job.in[row * job.ld + j] : 0u;
    }
    transpose_32x32_bits(x);
#pragma unroll
    for (int c = 0; c < 32; ++c) {
        const uint32_t row = 32u * j + c;
        if ((int64_t)row < job.cols) *reinterpret_cast<uint32_t *>(job.out + ((uint64_t)(2u * G + h) * job.out_rows + row) * 16u + 4u * i) = ~x[c];
    }
}

// A gradient's planes, with multipliers +-2^q: see MergeCode.
struct Gradient {
    const uint32_t *planes;
    int64_t plane_stride, ld;  // words
    int64_t M, N;
    MergeCode code;
    uint32_t *inexact;  // [kFlags]
};
// Whether the gradient holds a value that is not an E3M2 number, i.e. whose magnitude has set bits further than two apart.  On the
// planes' words as they lie, 32 elements at a time: u (or 2 u) minus a constant, bit by bit, its magnitude, and the pairs of its bits.
// Bound: memory (41 MB of planes in 10 us beside the transpositions).
__device__ __forceinline__ void look_over(const Gradient &a, const uint32_t block) {
    const uint32_t Nw = (uint32_t)((a.N + 31) / 32);
    const uint32_t minus = (uint32_t)(a.code.twice ? 2 * a.code.neg_sum - a.code.bias : a.code.neg_sum);
    uint32_t found = 0;
    for (uint64_t at = (uint64_t)block * 256u + threadIdx.x; at < (uint64_t)a.M * Nw; at += (uint64_t)kFlags * 256u) {
        const uint64_t m = at / Nw;
        const uint32_t j = (uint32_t)(at - m * Nw);
        uint32_t u[10];  // bits of u or 2 u
        u[8] = u[9] = 0u;
#pragma unroll
        for (int q = 0; q < 8; ++q) u[q] = (a.code.src[q] >= 0 ? a.planes[a.code.src[q] * a.plane_stride + (int64_t)m * a.ld + j] : 0u) ^ a.code.inv[q];
        if (a.code.twice) {
#pragma unroll
            for (int q = 8; q > 0; --q) u[q] = u[q - 1];
            u[0] = 0u;
        }
        uint32_t borrow = 0;
#pragma unroll
        for (int q = 0; q < 10; ++q) {
            const uint32_t c = 0u - ((minus >> q) & 1u), b = borrow;
            borrow = (~u[q] & (c | b)) | (c & b);
            u[q] ^= c ^ b;
        }
        const uint32_t sign = u[9];
        uint32_t carry = sign, below[8], wide = 0, seen = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {  // (the magnitude is at most 128)
            const uint32_t b = u[q] ^ sign;
            u[q] = b ^ carry;
            carry &= b;
            below[q] = seen |= u[q];
            if (q >= 3) wide |= u[q] & below[q - 3];
        }
        const int64_t left = a.N - 32 * (int64_t)j;
        found |= left >= 32 ? wide : wide & ((1u << left) - 1u);
    }
    const int any = __syncthreads_or((int)found);
    if (threadIdx.x == 0) a.inexact[block] = any ? 1u : 0u;
}

// The first launch of a backward step: both bits images, and the look at the gradient.  Bound: the transpositions' latency (one load,
// 300 instructions and one store phase), under which the look's memory traffic goes.
__global__ __launch_bounds__(256) void transpose_to_image_kernel(const Gradient a, const BitsJob w, const BitsJob x) {
    uint32_t block = blockIdx.x;
    if (block < w.blocks) {
        transpose_to_image(w, block);
    } else if ((block -= w.blocks) < x.blocks) {
        transpose_to_image(x, block);
    } else {
        look_over(a, block - x.blocks);
    }
}

__device__ __forceinline__ uint32_t add_bytes(uint32_t x, uint32_t y) {  // byte-wise sum mod 256
    return ((x & 0x7F7F7F7Fu) + (y & 0x7F7F7F7Fu)) ^ ((x ^ y) & 0x80808080u);
}
// One row's 32 elements word .. + 31 (signed bytes) into a values image
struct Image {
    uint8_t *base;
    uint32_t rows, groups, halves;  // rows of a group; groups of 256, of 128 (int8)
};
__device__ __forceinline__ void put(const Image &im, const bool as_bytes, const uint32_t G, const uint32_t c, const uint32_t row, const uint32_t (&bytes)[8]) {
    if (as_bytes) {
        if (2u * G + (c >> 2) >= im.halves) return;  // (a half group of zeros at the end, which is not multiplied)
        uint32_t o[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // elements 0 2 4 6 1 3 5 7
            o[2 * q] = __builtin_amdgcn_perm(bytes[2 * q + 1], bytes[2 * q], 0x06040200u);
            o[2 * q + 1] = __builtin_amdgcn_perm(bytes[2 * q + 1], bytes[2 * q], 0x07050301u);
        }
        uint8_t *const at = im.base + ((uint64_t)(2u * G + (c >> 2)) * im.rows + row) * 128u;
        const uint32_t turn = (row >> 1) & 7u, p = 2u * (c & 3u);
        *reinterpret_cast<uint4 *>(at + 16u * (p ^ turn)) = make_uint4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<uint4 *>(at + 16u * ((p + 1u) ^ turn)) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
        typedef float v16f __attribute__((ext_vector_type(16)));
        v16f even, odd;
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) (e & 1 ? odd : even)[2 * q + (e >> 1)] = (float)(int8_t)(bytes[q] >> (8 * e));
        const v6u f = __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(even, odd, 16.0f);  // (interleaves its operands; units of 1/16)
        uint8_t *const high = im.base + (uint64_t)im.groups * im.rows * 128u;
        *reinterpret_cast<uint4 *>(im.base + ((uint64_t)G * im.rows + row) * 128u + 16u * (c ^ ((row >> 1) & 7u))) = make_uint4(f[0], f[1], f[2], f[3]);
        *reinterpret_cast<uint2 *>(high + (((uint64_t)G * 4u + (c & 3u)) * im.rows + row) * 16u + 8u * ((c >> 2) ^ ((row >> 4) & 1u))) = make_uint2(f[4], f[5]);
    }
}

// Both values images of a gradient at once: rows m with k = n (out) and rows n with k = m (out_t).
// A workgroup takes 128 rows x 256 columns (one group of out, half a group of out_t), a thread four rows x one word: the planes' words
// become 32 bytes per row (bit-matrix transposition in registers), which the conversion instruction packs for out; 4 x 4 byte
// transpositions turn four rows' bytes into dwords along m, and LDS collects those to 32 bytes per column for out_t.  LDS: column n at
// dword 36 n, its dwords rotated by 8 (n / 32 mod 4) and moved on by 32 for the upper half, so that the 64 dword writes of a wave (eight
// words x eight row groups) fall on 64 banks.  The 16-byte reads of a column's pieces meet in twos (36 dwords a column): half of the LDS
// cycles at 10000 x 4096.
__global__ __launch_bounds__(256) void merge_transpose_kernel(const Gradient a, const Image out, const Image out_t) {
    constexpr int kPitch = 36;
    __shared__ __attribute__((aligned(16))) uint32_t s_t[256 * kPitch + 32];
    const uint32_t t = threadIdx.x, j = t & 7u, rg = t >> 3, G = blockIdx.x, Gt = blockIdx.y >> 1, h = blockIdx.y & 1u;
    const int64_t m0 = (int64_t)blockIdx.y * 128, jw = (int64_t)G * 8 + j, Nw = (a.N + 31) / 32;
    uint32_t o[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = m0 + 4 * rg + i;
        const bool in = m < a.M && jw < Nw;
#pragma unroll
        for (int q = 0; q < 8; ++q) o[i][q] = (in && a.code.src[q] >= 0) ? a.planes[a.code.src[q] * a.plane_stride + m * a.ld + jw] : 0u;
    }
    static_assert(kFlags == 512, "two words a thread");
    const bool as_bytes = __syncthreads_or((int)(a.inexact[t] | a.inexact[t + 256u])) != 0;
    const uint32_t minus = (uint32_t)((-a.code.neg_sum) & 0xFF) * 0x01010101u, bias = (uint32_t)(a.code.bias & 0xFF) * 0x01010101u;
    const int64_t left = a.N - 32 * jw;  // columns of this word that exist
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = m0 + 4 * rg + i;
        uint32_t r8[8], v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r8[q] = o[i][q] ^ a.code.inv[q];
        join_32_codes(r8, v);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v[q] = add_bytes(v[q], minus);
            if (a.code.twice) v[q] = add_bytes(add_bytes(v[q], v[q]), bias);
        }
        if (m >= a.M || left < 32) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t have = m < a.M ? left - 4 * q : 0;
                v[q] &= have >= 4 ? 0xFFFFFFFFu : (have <= 0 ? 0u : (1u << (8 * (int)have)) - 1u);
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) o[i][q] = v[q];
        if (m < a.M) put(out, as_bytes, G, j, (uint32_t)m, v);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint32_t rows[4] = {o[0][q], o[1][q], o[2][q], o[3][q]};
        uint32_t cols[4];
        transpose_4x4_bytes(rows, cols);
#pragma unroll
        for (int p = 0; p < 4; ++p) s_t[(32 * j + 4 * q + p) * kPitch + ((rg + 8 * (j & 3)) & 31) + 32 * (j >> 2)] = cols[p];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
        const uint32_t idx = t + 256u * u, nl = idx >> 2, pc = idx & 3u, jn = nl >> 5;
        const int64_t n = (int64_t)G * 256 + nl;
        const uint4 *const p = reinterpret_cast<const uint4 *>(&s_t[nl * kPitch + ((8 * pc + 8 * (jn & 3)) & 31) + 32 * (jn >> 2)]);
        const uint4 x = p[0], y = p[1];
        const uint32_t v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        if (n < a.N) put(out_t, as_bytes, Gt, 4u * h + pc, (uint32_t)n, v);
    }
}

// Sizes of images.  A group has as many rows as the operand, rounded up to whole lines: what a tile reads beyond them belongs to the group
// behind it, or is the room left behind the last one.  (Groups of whole tiles took up to 255 rows more each, and eight planes of a
// transposed gradient then no longer fitted the workspace that holds them as planes.)
uint32_t padded(int64_t rows) { return (uint32_t)(ceil_div(rows, 8) * 8); }
constexpr int kGroupK = 256;
uint32_t groups_of(int64_t k) { return (uint32_t)ceil_div(k, kGroupK); }
uint32_t halves_of(int64_t k) { return k <= kGroupK / 2 ? 2u : (uint32_t)ceil_div(k, kGroupK / 2); }  // at least two (the kernel relies on it)
size_t beyond(int64_t rows, int64_t tile) { return (size_t)(ceil_div(rows, tile) * tile - padded(rows)); }  // rows a last tile reads
// int8: 128 bytes a row and half group, FP6: 192 a row and group
size_t values_bytes(int64_t rows, int64_t k) {
    const size_t as_bytes = (size_t)halves_of(k) * 128, as_fp6 = (size_t)groups_of(k) * 192;
    return (as_bytes > as_fp6 ? as_bytes : as_fp6) * padded(rows) + beyond(rows, 128) * 128;
}
size_t bits_bytes(int64_t rows, int64_t k) { return (size_t)groups_of(k) * padded(rows) * (kGroupK / 8) + beyond(rows, 256) * 16; }

// Tiles of 128 x 256 or 128 x 128, two workgroups on a compute unit, by the time of their rounds (us per group of k, with two and with one
// workgroup on a unit; FP6: 10000 x 4096 x 4096, 1264 and 2528 tiles, 93 against 109 us, 1000 x 4096 x 4096, 128 and 256, 22.2 against 17.4;
// 256 x 256 on one workgroup of eight waves, 640 and 64 tiles, 107 and 31).
struct Tiles {
    bool wide;
    double us;  // per group, int8
    Tiles(int64_t M, int64_t N, int64_t cus) {
        auto rounds = [cus](int64_t tiles, double two, double one) {
            const int64_t rest = tiles % (2 * cus);
            return (double)(tiles / (2 * cus)) * two + (rest == 0 ? 0.0 : (rest <= cus ? one : two));
        };
        const int64_t tiles_m = ceil_div(M, 128), w = tiles_m * ceil_div(N, 256), n = tiles_m * ceil_div(N, 128);
        wide = rounds(w, 2.0, 1.3) <= rounds(n, 1.22, 1.0);
        us = wide ? rounds(w, 3.26, 1.75) : rounds(n, 2.0, 1.36);
    }
};

// C = alpha S of a values image (M rows) and a bits image (N rows) over K elements
int launch_product(const uint8_t *a, const uint8_t *w, const uint32_t *inexact, int32_t *C, int64_t ldc, int64_t M, int64_t N, int64_t K, int32_t alpha,
                   hipStream_t s) {
    GemmArgs g;
    MixedArgs x;
    std::memset(&g, 0, sizeof(g));
    g.M = M, g.N = N, g.K = K, g.epi.C = C, g.epi.ldc = ldc;
    x.a = a, x.w = w, x.inexact = inexact, x.rows_a = padded(M), x.rows_w = padded(N), x.groups = groups_of(K), x.halves = halves_of(K);
    x.alpha = alpha, x.alpha_shift = -1;
    for (int sh = 0; sh < 31; ++sh)
        if (alpha == ((int64_t)1 << sh)) x.alpha_shift = sh;
    const int64_t cus = compute_units(), tiles_m = ceil_div(M, 128);
    const bool is_wide = Tiles(M, N, cus).wide;
    const int64_t total = tiles_m * ceil_div(N, is_wide ? 256 : 128);
    x.tiles = make_tiles(tiles_m, total / tiles_m);
    return QNN_LAUNCH("gemm_mixed", (is_wide ? gemm_mixed_kernel<4, 2, 4, 2> : gemm_mixed_kernel<4, 2, 2, 2>), dim3((unsigned)(total < 2 * cus ? total : 2 * cus)),
                      dim3(256), 0, s, g, x);
}

}  // namespace

// Whether every sum of the products stays exact: values up to 128 times +-1, float sums within 2^24 (and 2 alpha within 32 bits).
static bool in_range(const Planes &pl, const MergeCode &c, int64_t longest) {
    int64_t hi = 0, lo = 0;
    for (int p = 0; p < pl.count; ++p) {
        const int64_t d = pl.coef[p] / c.scale, ad = d < 0 ? -d : d;
        if (pl.mode == QNN_PLANE_BIT)
            (d > 0 ? hi : lo) += ad;
        else
            hi += ad, lo += ad;
    }
    return (hi > lo ? hi : lo) * longest <= (1 << 24) && c.scale <= (1 << 29);
}

bool backward_supports(const BackwardArgs &b) {
    MergeCode c;
    if (!merge_code(b.pg, c)) return false;
    const int64_t longest = b.M > b.N ? b.M : b.N;
    return in_range(b.pg, c, longest) && b.M <= 0x7FFFFE00 && b.N <= 0x7FFFFE00 && b.K <= 0x7FFFFE00 &&
           ceil_div(b.M, 128) * ceil_div(b.K, 128) <= 0x7FFFFFFF && ceil_div(b.N, 128) * ceil_div(b.K, 128) <= 0x7FFFFFFF && ceil_div(b.M, 256) <= 32767;
}

// (four launches and temporary memory from the pool cost the host 38 us at least)
double backward_us(const BackwardArgs &b) {
    const int64_t cus = compute_units();
    const double prepare = 16.0 + 0.95e-6 * (double)b.M * (double)b.N, store = 0.35e-6 * (double)(b.M + b.N) * (double)b.K;
    const double products = 7.0 + groups_of(b.N) * Tiles(b.M, b.K, cus).us + groups_of(b.M) * Tiles(b.N, b.K, cus).us;
    return prepare + products + store < 38.0 ? 38.0 : prepare + products + store;
}

int launch_backward(const BackwardArgs &b, void *workspace, size_t workspace_bytes, bool &no_memory, hipStream_t s) {
    // images: the gradient in both orders, weights and activations transposed; what the workspace does not hold comes from the pool
    constexpr int kParts = 5;
    const size_t sizes[kParts] = {kFlags * 4, values_bytes(b.N, b.M), values_bytes(b.M, b.N), bits_bytes(b.K, b.N), bits_bytes(b.K, b.M)};
    size_t at[kParts], used = 0, borrowed = 0;
    bool in_pool[kParts];
    for (int i = 0; i < kParts; ++i) {
        in_pool[i] = used + sizes[i] > workspace_bytes;
        size_t &end = in_pool[i] ? borrowed : used;
        at[i] = end;
        end += sizes[i];
    }
    PoolMemory mem(s);
    no_memory = false;
    if (borrowed) {
        const int taken = mem.take(borrowed);
        no_memory = taken != QNN_OK;
        if (no_memory) return taken;
    }
    uint8_t *part[kParts];
    for (int i = 0; i < kParts; ++i) part[i] = static_cast<uint8_t *>(in_pool[i] ? mem.ptr : workspace) + at[i];

    BitsJob w, x;
    w.in = b.W, w.rows = b.N, w.cols = b.K, w.ld = b.ldw, w.out = part[3], w.out_rows = padded(b.K), w.groups = groups_of(b.N);
    x.in = b.A, x.rows = b.M, x.cols = b.K, x.ld = b.lda, x.out = part[4], x.out_rows = padded(b.K), x.groups = groups_of(b.M);
    w.blocks = w.groups * (uint32_t)ceil_div(b.K, 1024), x.blocks = x.groups * (uint32_t)ceil_div(b.K, 1024);
    Gradient g;
    merge_code(b.pg, g.code);
    g.planes = b.G, g.plane_stride = b.strideG, g.ld = b.ldg, g.M = b.M, g.N = b.N, g.inexact = reinterpret_cast<uint32_t *>(part[0]);
    const Image out = {part[2], padded(b.M), groups_of(b.N), halves_of(b.N)}, out_t = {part[1], padded(b.N), groups_of(b.M), halves_of(b.M)};
    const int32_t alpha = (int32_t)g.code.scale;
    int rc = QNN_LAUNCH("transpose_to_image", transpose_to_image_kernel, dim3(w.blocks + x.blocks + kFlags), dim3(256), 0, s, g, w, x);
    if (rc == QNN_OK) rc = QNN_LAUNCH("merge_transpose", merge_transpose_kernel, dim3(out.groups, 2u * out_t.groups), dim3(256), 0, s, g, out, out_t);
    if (rc == QNN_OK) rc = launch_product(part[2], part[3], g.inexact, b.gA, b.ld_ga, b.M, b.K, b.N, alpha, s);
    if (rc == QNN_OK) rc = launch_product(part[1], part[4], g.inexact, b.gW, b.ld_gw, b.N, b.K, b.M, alpha, s);
    return mem.give_back(rc);
}

}  // namespace mixed
}  // namespace qnn
