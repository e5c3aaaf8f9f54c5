// Internal declarations shared by the translation units of libqnn (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "qnn.h"

namespace qnn {

// Records the message returned by qnn_last_error() for the calling thread and passes `code` through.
int fail(int code, const char *fmt, ...);
// Records the engine that a call used (qnn_last_engine, qnn_last_engines) where it does not go through the common dispatch.
void note_engine(int engine);
// Checks hipGetLastError() after a launch; QNN_OK or QNN_ERR_HIP.
int check_launch(const char *what);
// Launches a kernel and reports the outcome of THIS launch: an error that an earlier HIP call of the caller left behind
// on the thread is discarded first, so that it is not blamed on a kernel that was in fact enqueued.
template <typename... KArgs, typename... Args>
inline int launch_checked(const char *what, void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned shmem,
                          hipStream_t stream, Args &&...args) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel, grid, block, shmem, stream, static_cast<KArgs>(args)...);
    return check_launch(what);
}
#define QNN_LAUNCH(what, ...) ::qnn::launch_checked(what, __VA_ARGS__)

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline int64_t words_for(int64_t K) { return (K + 31) / 32; }

// How the rows of the left operand are found in memory.  rows_are_pixels == 0: row m, word j is at
// base + m * ld + j (a plain packed matrix).  rows_are_pixels == 1: row m is output pixel (b, y, x) of a
// convolution over a channels-last packed image and word j = tap * Cw + c addresses channel word c of input pixel
// (y * stride + ky - pad, x * stride + kx - pad); taps that fall outside the image read as zero words.
struct LeftAddr {
    const uint32_t *base;
    int64_t ld;            // words between consecutive rows (matrix) -- unused for pixels
    int64_t plane_stride;  // words between consecutive planes
    int rows_are_pixels;
    int rows_are_bytes;  // matrix-core engine only: base points at uint8 codes, one per element, ld = row pitch in bytes
    int H, Wd, Ho, Wo, Cw, KH, KW, pad, stride;
};

// One multi-plane operand description passed by value to the kernels.
struct Planes {
    int count;
    int mode;  // qnn_plane_mode
    int32_t coef[QNN_MAX_PLANES];
};

// What the multiply writes.  T == nullptr: int32 sums to C (leading dimension ldc).
// T != nullptr: bit = (sum >= T[n]) xor flip[n], packed along n into out_bits (leading dimension ldo words).
struct Epilogue {
    int32_t *C;
    int64_t ldc;
    const int32_t *T;
    const uint8_t *flip;
    uint32_t *out_bits;
    int64_t ldo;
};

struct GemmArgs {
    LeftAddr A;
    Planes pa;
    const uint32_t *W;
    int64_t ldw;
    int64_t strideW;
    Planes pw;
    Epilogue epi;
    int64_t M, N, K;  // K = true number of elements per row (not words)
    int64_t Kw;       // words per row = ceil(K/32) (for pixels: KH*KW*Cw)
    // Right operand of int8 values instead of planes (left operand: rows_are_bytes too): row pitch ld_w_bytes, a multiple of 128
    const int8_t *w_bytes;
    int64_t ld_w_bytes;
    // Optional, with a left operand of uint8 codes only: the +-1 weights as the image of qnn_gemm_codes.hip and 128 * (sum of the
    // weights of row n), both written by codes::launch_weight_image earlier on the same stream.  Null: the kernels expand the packed bits.
    const uint32_t *w_image;
    const int32_t *rw_scaled;
    // Only for convolutions of +-1 maps (gemm_map_kernel): class_thr[cls * class_ld + n] is the threshold of filter n for a pixel
    // of border class cls (bit 0: first row, 1: last row, 2: first column, 3: last column).
    const int32_t *class_thr;
    int64_t class_ld;
    const uint32_t *pool_and;  // +-1 maps: 2 x 2 max-pooling follows; packed flags of the filters whose bits are AND-ed
    uint32_t pool_invert;      // ... inverted with this
};

// Tile index with consecutive ids of one XCD (ids congruent mod 8 share an L2) laid on neighbouring tiles, and tiles
// walked in bands of 8 tile-rows so that the W panels a band needs stay cached.
__device__ __forceinline__ void tile_of_block(uint32_t bid, uint32_t total, uint32_t tiles_m, uint32_t tiles_n,
                                              uint32_t &tm, uint32_t &tn) {
    const uint32_t xcd = bid & 7u, slot = bid >> 3;
    const uint32_t q = total >> 3, r = total & 7u;
    const uint32_t id = xcd * q + (xcd < r ? xcd : r) + slot;
    constexpr uint32_t kBand = 8;
    const uint32_t per_band = kBand * tiles_n;
    const uint32_t band = id / per_band;
    const uint32_t first_m = band * kBand;
    const uint32_t band_rows = (tiles_m - first_m < kBand) ? (tiles_m - first_m) : kBand;
    const uint32_t in_band = id - band * per_band;
    tm = first_m + in_band % band_rows;
    // Tiles that run at the same time sit at the same position of different bands.  Rotating the columns band by band
    // keeps them in different column ranges of C, so that their stores (and W reads) go to different memory channels
    // even when the row pitch of C is a power of two.
    tn = (in_band / band_rows + band * 4u) % tiles_n;
}

// a / d and the remainder for a < 2^31 (the product with floor(2^32 / d) falls short by less than one)
__device__ __forceinline__ uint32_t quotient(const uint32_t a, const uint32_t d, const uint32_t inv, uint32_t &rem) {
    uint32_t q = __umulhi(a, inv);
    rem = a - q * d;
    if (rem >= d) ++q, rem -= d;
    return q;
}
// floor(2^32 / d) for quotient, 2^32 - 1 for 1
static inline uint32_t inverse_of(int64_t d) { return d > 1 ? (uint32_t)(4294967296LL / d) : 0xFFFFFFFFu; }

// The same tile order without divisions by numbers that only the host knows in advance, three of which cost a workgroup some 0.4 us before its first
// load (1000 x 1000 x 1000 5.3 -> 5.0 us).
struct Tiles {
    uint32_t m, n, total, inv_band, inv_n, last_rows, inv_last;  // last_rows: tile rows of the last band
};
static inline Tiles make_tiles(int64_t m, int64_t n) {
    const int64_t last = m % 8 ? m % 8 : 8;
    return Tiles{(uint32_t)m, (uint32_t)n, (uint32_t)(m * n), inverse_of(8 * n), inverse_of(n), (uint32_t)last, inverse_of(last)};
}
__device__ __forceinline__ void tile_of_block(const uint32_t bid, const Tiles &t, uint32_t &tm, uint32_t &tn) {
    const uint32_t xcd = bid & 7u, slot = bid >> 3, q = t.total >> 3, r = t.total & 7u;
    uint32_t in_band, row;
    const uint32_t band = quotient(xcd * q + (xcd < r ? xcd : r) + slot, 8u * t.n, t.inv_band, in_band);
    uint32_t col = in_band >> 3;
    row = in_band & 7u;
    if (8u * band + 8u > t.m) col = quotient(in_band, t.last_rows, t.inv_last, row);
    tm = 8u * band + row;
    (void)quotient(col + band * 4u, t.n, t.inv_n, tn);
}

// Engines.  Both return QNN_OK / QNN_ERR_*; `mfma_supports` says whether the matrix-core engine can take the job.
int launch_gemm_valu(const GemmArgs &g, hipStream_t s);
bool valu_supports(const GemmArgs &g);
bool mfma_supports(const GemmArgs &g, bool fp4 = false);  // fp4: on the FP4 (E2M1) matrix-core path
bool mfma_preferred(const GemmArgs &g);  // whether AUTO should pick it for this shape
int launch_gemm_mfma(const GemmArgs &g, hipStream_t s, bool fp4 = false);
// The same engine's kernel for operands of several bit planes, which expands them once per workgroup into LDS.
bool stage_supports(const GemmArgs &g);
double stage_us(const GemmArgs &g);  // about how long it takes there (microseconds)
int compute_units();
int launch_gemm_stage(const GemmArgs &g, hipStream_t s);
// FP4 matrix-core kernels for products of any size and layout (qnn_gemm_slice.hip: small tiles whose waves share k;
// qnn_gemm_tile.hip: larger tiles).  slice_preferred: whether they take the product and beat the engine (`route`) that the shape
// would go to otherwise; launch_gemm_slice chooses between the two.
bool slice_preferred(const GemmArgs &g, int route);
double slice_us(const GemmArgs &g);  // about how long it takes there (microseconds; 1e30 if not taken)
int launch_gemm_slice(const GemmArgs &g, hipStream_t s);
int launch_gemm_tile(const GemmArgs &g, hipStream_t s);
// Both products of the backward step from FP6 gradients (g_a = g W into gA, g_W = g^T a into gW): whether they take this way, and the
// launches (qnn_gemm_mixed.hip).  no_memory: the stream's pool could not supply what the workspace does not hold; nothing has
// been launched then.
struct BackwardArgs {
    Planes pg;
    const uint32_t *G, *W, *A;
    int64_t ldg, strideG, ldw, lda;
    int32_t *gA, *gW;
    int64_t ld_ga, ld_gw, M, N, K;
};
bool backward_mixed_preferred(const BackwardArgs &b);
namespace mixed {
bool backward_supports(const BackwardArgs &b);
double backward_us(const BackwardArgs &b);  // about how long it takes (microseconds) where the gradient is int8
int launch_backward(const BackwardArgs &b, void *workspace, size_t workspace_bytes, bool &no_memory, hipStream_t s);
}
bool panel_takes(const GemmArgs &g);  // whether the FP4 route would use the panel-fed kernel (on rows that it pays for: 1999 x 3001 x 300 7.0 us on tiles, 8.2 on panels)
void panel_shape(int64_t M, int64_t N, int64_t Kw, int &shape, int &per);  // ... a +-1 map with which tiles (panel::Shape)

// How planes with multipliers +-2^q stand for a byte: the plane of bit q (-1: none), its inversion; value = scale ((sum 2^q bit -
// neg_sum) [* 2 + bias]), the number in brackets within int8.
struct MergeCode {
    int src[8];
    uint32_t inv[8];
    int32_t neg_sum, bias;
    int twice;
    int64_t scale;
};
bool merge_code(const Planes &pl, MergeCode &c);  // false: other multipliers, or values beyond int8

// Temporary device memory from the stream's pool, given back in stream order.
struct PoolMemory {
    void *ptr = nullptr;
    hipStream_t s;
    explicit PoolMemory(hipStream_t stream) : s(stream) {}
    int take(size_t bytes) {
        if (hipMallocAsync(&ptr, bytes, s) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            ptr = nullptr;
            return fail(QNN_ERR_HIP, "gemm: no memory for the merged operands (%zu bytes)", bytes);
        }
        return QNN_OK;
    }
    int give_back(int rc) {
        if (ptr && hipFreeAsync(ptr, s) != hipSuccess) {
            (void)hipGetLastError();
            if (rc == QNN_OK) rc = fail(QNN_ERR_HIP, "gemm: returning the merged operands' memory failed");
        }
        return rc;
    }
};

// Products of uint8 codes and +-1 weights that stay bits (qnn_gemm_codes.hip), threshold output: w_image (image_bytes(N, K) bytes) and
// rw_scaled (N words) of the arguments are written by launch_weight_image, earlier on the same stream.
namespace codes {
size_t image_bytes(int64_t N, int64_t K);
bool supports(const GemmArgs &g);
int launch_weight_image(const GemmArgs &g, hipStream_t s);
// ... few rows, without an image (codes and rows on 16-byte boundaries)
bool small_preferred(const GemmArgs &g, bool large, bool has_image);  // large: codes would be multiplied otherwise too, with an image of the weights or without
int launch_small(const GemmArgs &g, hipStream_t s);
int launch(const GemmArgs &g, hipStream_t s);
}  // namespace codes

// Operands of the int8 kernel.
namespace bytes_panel {
// Bit planes of both operands of `g` merged to one int8 per element (rows of ld_out bytes, a multiple of 128, zeros
// beyond K): value = scale_of_operand * int8, and `scale` returns the product of the two operands' factors.
// merge_supports: whether the values of both operands fit int8.
bool merge_supports(const Planes &pa, const Planes &pw);
int launch_merge_planes(const GemmArgs &g, int8_t *outA, int8_t *outW, int64_t ld_out, int64_t &scale, hipStream_t s);
}
int launch_pack_sign(const float *x, int64_t rows, int64_t K, int64_t ldx, uint32_t *out, int64_t ldo, hipStream_t s);
int launch_pack_bitplanes(const uint8_t *v, int64_t rows, int64_t K, int64_t ldv, int nbits, uint32_t *planes,
                          int64_t ld, int64_t plane_stride, hipStream_t s);
int launch_threshold_sign(const int32_t *C, int64_t ldc, int64_t M, int64_t N, const int32_t *T, const uint8_t *flip,
                          uint32_t *out, int64_t ldo, hipStream_t s);

// 3 x 3 "same" convolution of a +-1 feature map (held as its plane "value is -1", [B][H][Wd][ceil(C / 32)] words) with +-1 filters
// and threshold output, on the panel-fed FP4 kernel.  bit = (conv >= T[n]) xor !flip_complement[n]: the caller passes the COMPLEMENT of
// its flip flags.  class_thr (16 x conv_class_ld(N) words) is written beforehand, on the same stream, by
// launch_conv_first or launch_conv_class_thr (for all convolutions of a network at once).  The 2 x 2 max-pooling that follows is done along if
// conv_map_pools (pool_and = packed flip flags of the filters, pool_invert = the map holds inverted bits; null: no pooling).
bool conv_map_supports(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N);
bool conv_map_preferred(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N, bool in_lds, bool sliced);  // ... image::, slice::map_supports
bool conv_map_pools(int64_t H, int64_t Wd);
// The same convolution where tiles are few (qnn_gemm_slice.hip): thresholds as they are, flips not complemented.
namespace slice {
bool map_supports(int64_t B, int64_t H, int64_t Wd, int64_t C, int64_t N, bool pooled);
int launch_map(const uint32_t *plane, int64_t B, int H, int Wd, int64_t C, const uint32_t *W, int64_t N, const int32_t *T, const uint8_t *flip, uint32_t *out,
               int64_t ldo, const uint32_t *pool_and, bool pool_invert, hipStream_t s);
}  // namespace slice
int64_t conv_class_ld(int64_t N);
int launch_conv_map(const uint32_t *plane, int64_t B, int H, int Wd, int64_t C, const uint32_t *W, int64_t N, const uint8_t *flip_complement,
                    uint32_t *out, int64_t ldo, const int32_t *class_thr, const uint32_t *pool_and, bool pool_invert, hipStream_t s);
// The same by the kernel that holds a tile's pixels in LDS as operands (qnn_gemm_image.hip), which needs no class thresholds and pools maps of
// any size along; map_supports: whether a tile's pixels fit there.  ones (may be null): also writes the "inside the image" plane of the output.
namespace image {
bool map_supports(int64_t B, int64_t H, int64_t W, int64_t C, int64_t N, bool pooled);
int launch_map(const uint32_t *plane, int64_t B, int H, int W, int64_t C, const uint32_t *filters, int64_t N, const int32_t *T, const uint8_t *flip_complement,
               uint32_t *out, uint32_t *ones, int64_t ldo, const uint32_t *pool_and, bool pool_invert, hipStream_t s);
// ... and of an image of bit planes: whether the kernel takes the convolution, whether it is expected to be the fastest, the launch
bool conv_supports(const GemmArgs &g);
bool conv_preferred(const GemmArgs &g);
int launch_conv(const GemmArgs &g, hipStream_t s);
}  // namespace image
struct ConvPrepJobs {
    int count;
    const uint32_t *W[2 * QNN_MAX_LAYERS];  // [N][9][Cw] filter bits
    const int32_t *T[2 * QNN_MAX_LAYERS];
    int32_t *out[2 * QNN_MAX_LAYERS];       // [16][ld]
    int64_t N[2 * QNN_MAX_LAYERS], ld[2 * QNN_MAX_LAYERS];
    int Cw[2 * QNN_MAX_LAYERS];
    int64_t C[2 * QNN_MAX_LAYERS];          // channels
    int64_t first_block[2 * QNN_MAX_LAYERS + 1];  // filled by the launch
};
// Flip flags of the layers of a network, turned into packed words and inverted bytes
struct FlagJobs {
    int count;
    const uint8_t *flip[2 * QNN_MAX_LAYERS];  // may be null: no channel flipped
    int64_t n[2 * QNN_MAX_LAYERS];
    uint32_t *bits[2 * QNN_MAX_LAYERS];
    uint8_t *inv[2 * QNN_MAX_LAYERS];
};
// (the layers' flip flags in the same launch; either count may be 0)
int launch_conv_class_thr(const ConvPrepJobs &jobs, const FlagJobs &flags, hipStream_t s);

// First convolution of a ConvNet straight from a uint8 image with at most three channels (3 x 3, pad 1, stride 1,
// threshold output packed along the filters): whether the kernel takes the shape, and its launch.
bool conv_first_supports(int64_t C0, int64_t N, int KH, int KW, int pad, int stride);
// flip_all: every flip flag counts as its complement.  jobs, flags: prepared in the same launch, for later layers (counts may be 0).
// ones (may be null): also writes the "inside the image" plane of the output map, [pixels][ldo] like `out`.
int launch_conv_first(const uint8_t *x, int64_t B, int H, int Wd, int C0, const uint32_t *W, int64_t N, const int32_t *T,
                      const uint8_t *flip, bool flip_all, uint32_t *out, uint32_t *ones, int64_t ldo, const ConvPrepJobs &jobs,
                      const FlagJobs &flags, hipStream_t s);

// rows x Cw words to be filled with the first C bits of every row: a map's "inside the image" plane (rows = 0: nothing)
struct OnesJob {
    uint32_t *out;
    int64_t rows;
    int Cw, C;
};
// ones (may be null) receives the "inside the image" plane of the pooled map; later: the one of another map
int launch_pool_bits(const uint32_t *in, int64_t B, int H, int Wd, int Cw, const uint32_t *use_and, bool invert_all,
                     uint32_t *out, uint32_t *ones, int C, const OnesJob &later, hipStream_t s);
int launch_ones_plane(const OnesJob &job, hipStream_t s);

}  // namespace qnn
