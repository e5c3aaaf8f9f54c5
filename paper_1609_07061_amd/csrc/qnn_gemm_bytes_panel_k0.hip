// Instantiations of the panel-fed matrix-core kernel for byte operands and the kernels that make its operands: the
// expansion of packed +-1 weights, and the merge of bit planes to int8 values (see qnn_gemm_bytes_panel_kernel.h).
#include "qnn_bitsplit.h"
#include "qnn_gemm_bytes_panel_kernel.h"

namespace qnn {
namespace bytes_panel {

namespace {
// Expansion of packed +-1 weights to bytes: out[n][k] = +1 / -1 for k < K and 0 for K <= k < ld_out; rw_scaled[n] =
// 128 sum_k w[n][k] = 256 popcount(row n) - 128 K.  One wave per row, lane j takes words j, j + 64, ...
__global__ __launch_bounds__(256) void expand_weights_kernel(const uint32_t *__restrict__ W, int64_t N, int64_t K, int64_t ldw,
                                                             int8_t *__restrict__ out, int64_t ld_out, int32_t *__restrict__ rw_scaled) {
    const int lane = threadIdx.x & 63;
    const int64_t words_out = ld_out / 32;  // ld_out is a multiple of 128
    const int64_t Kw = (K + 31) / 32;
    for (int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); n < N; n += (int64_t)gridDim.x * 4) {
        int32_t pop = 0;
        for (int64_t j = lane; j < words_out; j += 64) {
            const uint32_t w = j < Kw ? W[n * ldw + j] : 0u;
            pop += (int32_t)__builtin_popcount(w);
            uint32_t o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t t4 = (w >> (4 * q)) & 0xFu;
                const uint32_t ones = (t4 * 0x00204081u) & 0x01010101u;  // bit i of t4 at byte i
                // +1 where the bit is set, -1 (0xFF) where it is clear and the element exists, 0 beyond K
                uint32_t v = ones | ((ones ^ 0x01010101u) * 0xFFu);
                const int64_t k0 = 32 * j + 4 * q;
                if (k0 + 4 > K) {
                    uint32_t keep = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (k0 + e < K) keep |= 0xFFu << (8 * e);
                    v &= keep;
                }
                o[q] = v;
            }
            uint4 *dst = reinterpret_cast<uint4 *>(out + n * ld_out + 32 * j);
            dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
            dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) pop += __shfl_xor(pop, d, 64);
        if (lane == 0) rw_scaled[n] = 256 * pop - 128 * (int32_t)K;
    }
}

// Bit planes merged to one int8 per element: out[r][k] = bias + sum_p mult[p] * bit_p(r, k) for k < K, 0 for
// K <= k < ld_out (a multiple of 128).  The host has checked that every value fits int8 and that the positive and the
// negative multipliers each add up to at most 255.  One thread per 32 elements.
//   General multipliers: a nibble of a plane word becomes four bytes of 0 / 1 with one multiplication, the planes'
//   contributions are summed as four bytes per register (positive and negative multipliers apart, no carries between
//   bytes), and positive - negative + bias is formed byte-wise.
//   Multipliers +-2^q with distinct q (`pow2`): the word of the plane with 2^q, inverted where its multiplier is negative, is
//   row q of an 8 x 32 bit matrix whose transpose holds, per element, the byte sum_q 2^q (b_q xor inv_q), which is the value
//   plus the sum of the negative multipliers' magnitudes (`neg_sum`, subtracted byte-wise); `twice` doubles that first
//   (sign-mode planes: 2 b - 1).  Half of the transposition falls away where no plane is above 2^3 (`low`).
// Bound: the latency of one load and one store per thread and, behind a product, the drain of its stores (2240 and 4096 rows x 2048
// of 4 planes: 7.8 us behind a quantizer, 13 us behind a product of 37 MB).  Planes come from the host in the order of their powers, so
// that nothing is sorted here.
// Slot i of src, inv: the plane with 2^i (pow2) or plane i; -1: none.
struct MergeOperand {
    const uint32_t *planes;
    int64_t plane_stride, ld;  // words
    int64_t rows;
    int8_t *out;
    int32_t mult[QNN_MAX_PLANES];
    int32_t bias;
    int pow2, twice, low;
    int src[QNN_MAX_PLANES];
    uint32_t inv[QNN_MAX_PLANES];
    int32_t neg_sum;
};
__device__ __forceinline__ uint32_t add_bytes(uint32_t x, uint32_t y) {  // byte-wise sum mod 256
    return ((x & 0x7F7F7F7Fu) + (y & 0x7F7F7F7Fu)) ^ ((x ^ y) & 0x80808080u);
}
// word[q] bit c = bit q of code c  ->  codes[j] byte i = code 4 j + i (the inverse of split_32_codes: both of its
// stages are their own inverses)
__device__ __forceinline__ void join_32_codes(const uint32_t (&word)[8], uint32_t (&codes)[8]) {
    const uint32_t lo4[4] = {word[0], word[1], word[2], word[3]}, hi4[4] = {word[4], word[5], word[6], word[7]};
    uint32_t L[4], H[4];
    transpose_4x4_bytes(lo4, L);
    transpose_4x4_bytes(hi4, H);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        transpose_8x8_bits(L[g], H[g]);
        codes[2 * g] = L[g], codes[2 * g + 1] = H[g];
    }
}
// grid: x = groups of four rows, y = groups of 64 output words, z = operand
__global__ __launch_bounds__(256) void merge_planes_kernel(const MergeOperand a, const MergeOperand w, int64_t K, int64_t ld_out) {
    const MergeOperand &op = blockIdx.z == 0 ? a : w;
    const int64_t words_out = ld_out / 32, Kw = (K + 31) / 32;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), j = (int64_t)blockIdx.y * 64 + (threadIdx.x & 63);
    if (r >= op.rows || j >= words_out) return;
    // all planes' words first (independent loads), then the arithmetic
    uint32_t words[QNN_MAX_PLANES];
#pragma unroll
    for (int p = 0; p < QNN_MAX_PLANES; ++p)
        words[p] = ((op.src[p] >= 0 && j < Kw) ? op.planes[op.src[p] * op.plane_stride + r * op.ld + j] : 0u) ^ op.inv[p];
    uint32_t o[8];
    if (op.pow2) {
        if (op.low) {
            const uint32_t rows4[8] = {words[0], words[1], words[2], words[3], 0u, 0u, 0u, 0u};
            join_32_codes(rows4, o);
        } else {
            join_32_codes(words, o);
        }
        const uint32_t minus = (uint32_t)((-op.neg_sum) & 0xFF) * 0x01010101u;
        const uint32_t bias = (uint32_t)(op.bias & 0xFF) * 0x01010101u;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            uint32_t v = add_bytes(o[q], minus);
            if (op.twice) v = add_bytes(add_bytes(v, v), bias);
            o[q] = v;
        }
    } else {
        uint32_t pos[8], neg[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) pos[q] = 0u, neg[q] = 0u;
#pragma unroll
        for (int p = 0; p < QNN_MAX_PLANES; ++p) {
            if (op.src[p] < 0) break;
            const int32_t m = op.mult[p];
            const uint32_t am = (uint32_t)(m < 0 ? -m : m);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t ones = (((words[p] >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;  // bit i of the nibble at byte i
                if (m < 0)
                    neg[q] += ones * am;
                else
                    pos[q] += ones * am;
            }
        }
        const uint32_t bias1 = (uint32_t)((op.bias + 1) & 0xFF) * 0x01010101u;
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = add_bytes(add_bytes(pos[q], ~neg[q]), bias1);  // pos + ~neg + 1 + bias
    }
    if (32 * j + 32 > K) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t k0 = 32 * j + 4 * q;
            uint32_t keep = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k0 + e < K) keep |= 0xFFu << (8 * e);
            o[q] &= keep;
        }
    }
    uint4 *dst = reinterpret_cast<uint4 *>(op.out + r * ld_out + 32 * j);
    dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
    dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
}

// Both byte forms of a gradient at once, for the two products of the backward step: out[m][n] (rows of ld_out bytes) and
// out_t[n][m] (rows of ld_t), with the sums of every row and column added to row_sums / col_sums.  Planes as in
// merge_planes_kernel with multipliers +-2^q: src[q] is the plane that holds bit q (-1: none), inv[q] its inversion.
// Bound: memory (a byte is written twice and one bit per plane read once).  A workgroup takes 128 rows x 256 columns, a thread four
// rows x one word: the planes' words become 32 bytes per row (bit-matrix transposition in registers), 4 x 4 byte transpositions
// turn four rows' bytes into dwords along m, and LDS collects those to 128 contiguous bytes per column.  LDS: column n at dword
// 36 n, its dwords rotated by 8 (n / 32 mod 4) and moved on by 32 for the upper half, so that the 64 dword writes of a wave (eight
// words x eight row groups) fall on 64 banks.
struct MergeBoth {
    const uint32_t *planes;
    int64_t plane_stride, ld;  // words
    int64_t M, N;
    int src[8];
    uint32_t inv[8];
    int32_t neg_sum, bias;
    int twice;
    int8_t *out, *out_t;
    int64_t ld_out, ld_t;
    int32_t *row_sums, *col_sums;
};
__global__ __launch_bounds__(256) void merge_transpose_kernel(const MergeBoth a) {
    constexpr int kPitch = 36;
    __shared__ __attribute__((aligned(16))) uint32_t s_t[256 * kPitch + 32];
    const int t = threadIdx.x, j = t & 7, rg = t >> 3;
    const int64_t m0 = (int64_t)blockIdx.y * 128, j0 = (int64_t)blockIdx.x * 8;
    const int64_t jw = j0 + j, Nw = (a.N + 31) / 32;
    uint32_t o[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = m0 + 4 * rg + i;
        const bool in = m < a.M && jw < Nw;
#pragma unroll
        for (int q = 0; q < 8; ++q) o[i][q] = (in && a.src[q] >= 0) ? a.planes[a.src[q] * a.plane_stride + m * a.ld + jw] : 0u;
    }
    const uint32_t minus = (uint32_t)((-a.neg_sum) & 0xFF) * 0x01010101u, bias = (uint32_t)(a.bias & 0xFF) * 0x01010101u;
    const int64_t left = a.N - 32 * jw;  // columns of this word that exist
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = m0 + 4 * rg + i;
        uint32_t r8[8], v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r8[q] = o[i][q] ^ a.inv[q];
        join_32_codes(r8, v);
        int32_t sum = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v[q] = add_bytes(v[q], minus);
            if (a.twice) v[q] = add_bytes(add_bytes(v[q], v[q]), bias);
        }
        if (m >= a.M || left < 32) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t have = m < a.M ? left - 4 * q : 0;
                v[q] &= have >= 4 ? 0xFFFFFFFFu : (have <= 0 ? 0u : (1u << (8 * (int)have)) - 1u);
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            sum = __builtin_amdgcn_sdot4((int)v[q], 0x01010101, sum, false);
            o[i][q] = v[q];
        }
        if (m < a.M && 32 * jw < a.ld_out) {
            uint4 *dst = reinterpret_cast<uint4 *>(a.out + m * a.ld_out + 32 * jw);
            dst[0] = make_uint4(v[0], v[1], v[2], v[3]);
            dst[1] = make_uint4(v[4], v[5], v[6], v[7]);
        }
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) sum += __shfl_xor(sum, d, 64);
        if (j == 0 && m < a.M) atomicAdd(&a.row_sums[m], sum);
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
    for (int u = 0; u < 8; ++u) {
        const int idx = t + 256 * u, nl = idx >> 3, pc = idx & 7, jn = nl >> 5;
        const int64_t n = 32 * j0 + nl;
        const uint4 x = *reinterpret_cast<const uint4 *>(&s_t[nl * kPitch + ((4 * pc + 8 * (jn & 3)) & 31) + 32 * (jn >> 2)]);
        int32_t sum = __builtin_amdgcn_sdot4((int)x.x, 0x01010101, 0, false);
        sum = __builtin_amdgcn_sdot4((int)x.y, 0x01010101, sum, false);
        sum = __builtin_amdgcn_sdot4((int)x.z, 0x01010101, sum, false);
        sum = __builtin_amdgcn_sdot4((int)x.w, 0x01010101, sum, false);
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) sum += __shfl_xor(sum, d, 64);
        if (n < a.N) {
            *reinterpret_cast<uint4 *>(a.out_t + n * a.ld_t + m0 + 16 * pc) = x;
            if (pc == 0) atomicAdd(&a.col_sums[n], sum);
        }
    }
}

// A packed bit matrix transposed to bytes 0 / 1: out[c][r] = bit (r, c) for r < rows, 0 for rows <= r < ld_out (a multiple of
// 128).  A thread takes four rows x one word: the words' bits s, s + 8, s + 16, s + 24 as bytes, a 4 x 4 byte transposition, and a
// wave stores 256 contiguous bytes of one output row per instruction.  Also clears n_clear words at `clear`.
__global__ __launch_bounds__(256) void transpose_to_bytes_kernel(const uint32_t *__restrict__ in, int64_t rows, int64_t cols, int64_t ld,
                                                                 uint8_t *__restrict__ out, int64_t ld_out, int32_t *__restrict__ clear,
                                                                 int64_t n_clear) {
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    for (int64_t i = block * 256 + threadIdx.x; i < n_clear; i += (int64_t)gridDim.x * gridDim.y * 256) clear[i] = 0;
    const int64_t j = (int64_t)blockIdx.y * 4 + (threadIdx.x >> 6), r = 4 * ((int64_t)blockIdx.x * 64 + (threadIdx.x & 63));
    if (j >= (cols + 31) / 32 || r >= ld_out) return;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = r + i < rows ? in[(r + i) * ld + j] : 0u;
    uint8_t *dst = out + 32 * j * ld_out + r;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        uint32_t b[4], c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = (w[i] >> s) & 0x01010101u;
        transpose_4x4_bytes(b, c);
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (32 * j + s + 8 * p < cols) *reinterpret_cast<uint32_t *>(dst + (int64_t)(s + 8 * p) * ld_out) = c[p];
    }
}

// Multipliers and bias of an operand's merge, and the factor `scale` with value = scale * (merged int8); false if the
// merged values do not fit int8.
bool merge_plan(const Planes &pl, MergeOperand &op, int64_t &scale) {
    int64_t gcd = 0;
    for (int p = 0; p < pl.count; ++p) {
        int64_t x = gcd, y = pl.coef[p] < 0 ? -(int64_t)pl.coef[p] : pl.coef[p];
        if (y == 0) return false;
        while (y) {
            const int64_t t = x % y;
            x = y;
            y = t;
        }
        gcd = x;
    }
    int64_t hi = 0, lo = 0, sum = 0;  // range of sum_p d_p b_p, and sum_p d_p
    for (int p = 0; p < pl.count; ++p) {
        const int64_t d = pl.coef[p] / gcd;
        (d > 0 ? hi : lo) += d;
        sum += d;
        op.mult[p] = (int32_t)(pl.mode == QNN_PLANE_BIT ? d : 2 * d);
    }
    for (int p = pl.count; p < QNN_MAX_PLANES; ++p) op.mult[p] = 0;
    if (pl.mode == QNN_PLANE_BIT) {
        op.bias = 0;
        if (hi > 127 || lo < -128) return false;
    } else {
        // sum_p d_p (2 b_p - 1)
        op.bias = (int32_t)-sum;
        if (hi - lo > 127) return false;  // largest magnitude: every plane at the sign of its coefficient
    }
    // multipliers +-2^q with distinct q: the transposing merge
    op.pow2 = 1, op.low = 1, op.twice = pl.mode != QNN_PLANE_BIT, op.neg_sum = (int32_t)-lo;
    for (int q = 0; q < QNN_MAX_PLANES; ++q) op.src[q] = -1, op.inv[q] = 0u;
    for (int p = 0; p < pl.count && op.pow2; ++p) {
        const int64_t d = pl.coef[p] / gcd, ad = d < 0 ? -d : d;
        int q = 0;
        while (((int64_t)1 << q) < ad) ++q;
        if (((int64_t)1 << q) != ad || q > 7 || op.src[q] >= 0) {
            op.pow2 = 0;
        } else {
            op.src[q] = p;
            op.inv[q] = d < 0 ? 0xFFFFFFFFu : 0u;
            if (q > 3) op.low = 0;
        }
    }
    if (!op.pow2)
        for (int p = 0; p < QNN_MAX_PLANES; ++p) op.src[p] = p < pl.count ? p : -1, op.inv[p] = 0u;
    scale = gcd;
    return true;
}

template <bool kCodes>
KernelFn kernel_of(bool tail, int blocks) {
    if (tail) return gemm_bytes_panel_kernel<kCodes, true, 4>;
    if (blocks == 4) return gemm_bytes_panel_kernel<kCodes, false, 4>;
    return blocks == 3 ? gemm_bytes_panel_kernel<kCodes, false, 3> : gemm_bytes_panel_kernel<kCodes, false, 2>;
}
}  // namespace

KernelFn kernel_values(bool tail, int blocks) { return kernel_of<false>(tail, blocks); }

bool merge_supports(const Planes &pa, const Planes &pw) {
    MergeOperand a, w;
    int64_t sa, sw;
    return merge_plan(pa, a, sa) && merge_plan(pw, w, sw);
}

int launch_merge_planes(const GemmArgs &g, int8_t *outA, int8_t *outW, int64_t ld_out, int64_t &scale, hipStream_t s) {
    MergeOperand a, w;
    int64_t sa, sw;
    if (!merge_plan(g.pa, a, sa) || !merge_plan(g.pw, w, sw)) return fail(QNN_ERR_UNSUPPORTED, "merged values do not fit int8");
    a.planes = g.A.base, a.plane_stride = g.A.plane_stride, a.ld = g.A.ld, a.rows = g.M, a.out = outA;
    w.planes = g.W, w.plane_stride = g.strideW, w.ld = g.ldw, w.rows = g.N, w.out = outW;
    scale = sa * sw;
    const int64_t row_groups = ceil_div(g.M > g.N ? g.M : g.N, 4), word_groups = ceil_div(ld_out / 32, 64);
    if (row_groups > 0x7FFFFFFFLL || word_groups > 65535) return fail(QNN_ERR_SHAPE, "merge: too many elements");
    return QNN_LAUNCH("merge_planes", merge_planes_kernel, dim3((unsigned)row_groups, (unsigned)word_groups, 2), dim3(256), 0, s, a, w,
                      g.K, ld_out);
}

bool merge_both_supports(const Planes &pl) {
    MergeOperand op;
    int64_t scale;
    return merge_plan(pl, op, scale) && op.pow2;
}

int launch_merge_transpose(const Planes &pl, const uint32_t *planes, int64_t plane_stride, int64_t ld, int64_t M, int64_t N, int8_t *out,
                           int64_t ld_out, int8_t *out_t, int64_t ld_t, int32_t *row_sums, int32_t *col_sums, int64_t &scale, hipStream_t s) {
    MergeOperand op;
    if (!merge_plan(pl, op, scale) || !op.pow2) return fail(QNN_ERR_UNSUPPORTED, "merged values do not fit int8");
    MergeBoth a;
    a.planes = planes, a.plane_stride = plane_stride, a.ld = ld, a.M = M, a.N = N;
    for (int q = 0; q < 8; ++q) a.src[q] = op.src[q], a.inv[q] = op.inv[q];
    a.neg_sum = op.neg_sum, a.bias = op.bias, a.twice = op.twice;
    a.out = out, a.ld_out = ld_out, a.out_t = out_t, a.ld_t = ld_t, a.row_sums = row_sums, a.col_sums = col_sums;
    const int64_t bx = ceil_div(ld_out, 256), by = ceil_div(ld_t, 128);
    if (bx > 0x7FFFFFFFLL || by > 65535) return fail(QNN_ERR_SHAPE, "merge: too many elements");
    return QNN_LAUNCH("merge_transpose", merge_transpose_kernel, dim3((unsigned)bx, (unsigned)by), dim3(256), 0, s, a);
}

int launch_transpose_to_bytes(const uint32_t *in, int64_t rows, int64_t cols, int64_t ld, uint8_t *out, int64_t ld_out, int32_t *clear,
                              int64_t n_clear, hipStream_t s) {
    const int64_t bx = ceil_div(ld_out, 256), by = ceil_div((cols + 31) / 32, 4);
    if (bx > 0x7FFFFFFFLL || by > 65535) return fail(QNN_ERR_SHAPE, "transpose: too many elements");
    return QNN_LAUNCH("transpose_to_bytes", transpose_to_bytes_kernel, dim3((unsigned)bx, (unsigned)by), dim3(256), 0, s, in, rows, cols, ld, out,
                      ld_out, clear, n_clear);
}

KernelFn kernel(bool tail, int blocks) { return kernel_of<true>(tail, blocks); }

int launch_expand_weights(const uint32_t *W, int64_t N, int64_t K, int64_t ldw, int8_t *out, int64_t ld_out, int32_t *rw_scaled,
                          hipStream_t s) {
    const int64_t blocks = ceil_div(N, 4);
    return QNN_LAUNCH("expand_weights", expand_weights_kernel, dim3((unsigned)(blocks > 4096 ? 4096 : blocks)), dim3(256), 0, s, W, N, K,
                      ldw, out, ld_out, rw_scaled);
}

}  // namespace bytes_panel
}  // namespace qnn
