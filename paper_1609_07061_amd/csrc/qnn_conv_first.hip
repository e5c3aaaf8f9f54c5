// First convolution of the binarized ConvNet (Alg. 4 on the network of App. A) straight from the 8-bit image.
//
// By Eq. (FirstLayer) the weighted plane products of a fixed-point input are x . w on the codes themselves.  With three
// input channels (or fewer) a 3 x 3 patch has at most 27 elements, so a pixel's whole patch is ONE operand row of
// v_mfma_i32_32x32x32_i8 (32 elements of k), the +-1 filters are the other operand, and a 32-pixel x 32-filter block of
// the layer is a single matrix-core instruction.  Going through bit planes instead (a packed word per pixel and plane
// that holds three bits, eight planes, nine taps) spends the machine on empty bits.
//   C[p][n] = sum_k (x[p][k] - 128) w[n][k] + 128 sum_k w[n][k],   k = (tap, channel), x = 0 outside the image
// (the second term per filter, formed once per workgroup), then bit = (C >= T[n]) xor flip[n], packed along n.
// A wave takes 32 consecutive pixels at a time: lane (r, kg) has sixteen patch bytes of pixel r in slots.  A row of the patch is 3 C0
// consecutive bytes of the image: slots 0 .. 8 hold the row above (kg = 0) or below (kg = 1), slots 9 .. 15 the first seven bytes of the
// middle row (kg = 0), slots 9 and 10 its last two (kg = 1).  So two loads bring a lane's bytes; what they bring too much meets zero
// weights.  For every block of 32 filters the wave reads its 16 filter bytes from LDS, negated, and thresholds, multiplies, and takes the
// signs of the 16 sums; the two lane halves are OR-ed into the pixel's output word.
#include <type_traits>

#include "qnn_gemm_mfma_kernel.h"
#include "qnn_internal.h"

namespace qnn {

namespace {

using mfma::or_halves;
using mfma::v16i;
using mfma::v4i;

constexpr int kFirstThreads = 256;
constexpr int kFirstMaxN = 1024;  // filters

// class_thr[cls][n] = floor(e / 2) as a float, clamped to +-2^23 (the sums it is compared with are far smaller), where
// e = 2 sum_{taps inside for cls} sum_c b[n][tap][c] - (taps inside) C - T[n] = (sum of the filter's weights on the taps
// inside) - T[n]: the convolution is that sum minus 2 S, S = sum_k p w, so it reaches T[n] iff S <= e / 2; cls bit 0: the pixel is in the first row (the upper taps lie outside), 1: last
// row, 2: first column, 3: last column.  Entries of filters beyond N are zero.  All layers of a network in one launch:
// sixteen lanes per filter, lane t < 9 counts the set bits of tap t, then lane c sums the taps that class c keeps.
// The first flag_blocks workgroups prepare the flip flags of the layers instead, as packed words and as inverted bytes (bits[w]
// bit t = (flip[32 w + t] != 0) for channels below n, flip == nullptr reading as all zero; inv[c] = !flip[c]); workgroup b takes
// channels 256 (b mod per_job) .. + 255 of layer b / per_job.
struct NetPrep {
    ConvPrepJobs jobs;
    FlagJobs flags;
    uint32_t flag_blocks, per_job, blocks;  // blocks: with those of the thresholds
};
static_assert(sizeof(NetPrep) <= 3840, "kernel arguments");
__device__ __forceinline__ void prepare_block(const NetPrep &p) {
    const ConvPrepJobs &jobs = p.jobs;
    const FlagJobs &flags = p.flags;
    if (blockIdx.x < p.flag_blocks) {
        const uint32_t fj = blockIdx.x / p.per_job;
        const uint8_t *flip = flags.flip[fj];
        const int64_t fn = flags.n[fj];
        const int lane = threadIdx.x & 63;
        const int64_t c = (int64_t)(blockIdx.x - fj * p.per_job) * 256 + threadIdx.x;
        if (c - lane >= fn) return;  // (whole waves leave: the ballot below sees complete waves only)
        const bool f = (c < fn && flip) ? (flip[c] != 0) : false;
        const unsigned long long m = __ballot(f);
        if (c < fn) flags.inv[fj][c] = f ? 0 : 1;
        const int64_t w = (c - lane) / 32;
        if (lane == 0) flags.bits[fj][w] = (uint32_t)m;
        if (lane == 32 && c < fn) flags.bits[fj][w + 1] = (uint32_t)(m >> 32);
        return;
    }
    const int64_t block = (int64_t)blockIdx.x - p.flag_blocks;
    int j = 0;
    while (j + 1 < jobs.count && block >= jobs.first_block[j + 1]) ++j;
    const int64_t n = (block - jobs.first_block[j]) * 16 + (threadIdx.x >> 4);
    const int sub = threadIdx.x & 15;
    const int64_t N = jobs.N[j], ld = jobs.ld[j];
    const int Cw = jobs.Cw[j];
    int32_t count = 0;
    if (n < N && sub < 9) {
        const uint32_t *w = jobs.W[j] + (n * 9 + sub) * Cw;
        for (int c = 0; c < Cw; ++c) count += __builtin_popcount(w[c]);
    }
    int64_t sum = 0, taps = 0;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const int32_t pc = __shfl(count, (threadIdx.x & 48) + tap, 64);  // (every lane takes part in the exchange)
        const int ky = tap / 3, kx = tap % 3;
        const bool outside = (ky == 0 && (sub & 1)) || (ky == 2 && (sub & 2)) || (kx == 0 && (sub & 4)) || (kx == 2 && (sub & 8));
        if (!outside) sum += pc, ++taps;
    }
    if (n < ld) {
        int64_t e = n < N ? 2 * sum - taps * jobs.C[j] - (int64_t)jobs.T[j][n] : 0;
        e >>= 1;  // floor
        e = e < -(1 << 23) ? -(1 << 23) : (e > (1 << 23) ? (1 << 23) : e);
        jobs.out[j][sub * ld + n] = (int32_t)__float_as_uint((float)(int32_t)e);
    }
}
__global__ __launch_bounds__(kFirstThreads) void conv_class_thr_kernel(const NetPrep p) { prepare_block(p); }

// n / d for n < 2^31: with l = ceil(log2 d), at least one, m = floor(2^(31 + l) / d) + 1 differs from 2^(31 + l) / d by at most 2^l / d
struct Divider {
    uint32_t m, shift, one;  // one: d = 1
    __device__ __forceinline__ uint32_t divide(uint32_t n) const { return one ? n : __umulhi(n, m) >> shift; }
};
Divider divider(uint32_t d) {
    uint32_t l = 1;
    while (((uint64_t)1 << l) < d) ++l;
    return {d == 1 ? 0u : (uint32_t)(((uint64_t)1 << (31 + l)) / d + 1), l - 1, d == 1 ? 1u : 0u};
}

struct FirstConvArgs {
    const uint8_t *x;     // [B][H][W][C0]
    const uint32_t *W;    // [N][9] words, bit c of word t = weight of tap t, channel c (set = +1)
    const int32_t *T;     // [N]
    const uint8_t *flip;  // [N] or null
    bool flip_all;        // every flip flag counts as its complement
    uint32_t *out;        // [B H W][ldo]
    uint32_t *ones;       // null, or [B H W][ldo]: receives the first N bits of every pixel set
    int64_t ldo;
    int64_t pixels;       // B H W
    int H, Wd, C0, N;
    Divider by_w, by_h;
};

// LDS: per filter 32 bytes and a threshold, per 32 filters a word of flip flags
constexpr size_t first_lds(int64_t padded) { return (size_t)padded * 36 + (size_t)padded / 8; }

// The first workgroups of the launch prepare what the later layers read: a launch of their own for it held up the first layer
// (App. A network, batch 4: 64.8 -> 62.2 us, batch 256: 144 -> 141.4 us).
// Bound: latency, of the filter tables at first and of a wave's two or three tiles then.  With a byte load per slot, a division per tile, and
// flip flags and thresholds applied to every sum it was vector instructions: 128 filters on 256 x 32 x 32 pixels 18.5 -> 12.3 us.
__global__ __launch_bounds__(kFirstThreads, 4) void conv_first_kernel(const FirstConvArgs a, const NetPrep prep) {
    if (blockIdx.x < prep.blocks) {
        prepare_block(prep);
        return;
    }
    const uint32_t block = blockIdx.x - prep.blocks, blocks = gridDim.x - prep.blocks;
    const uint32_t Npad = ((uint32_t)a.N + 31u) / 32u * 32u, Nw = Npad / 32u;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t *const sW = lds;
    // threshold - 1 - 128 sum_k w: the matrix-core sum S meets the threshold iff S > that
    int32_t *const sE = reinterpret_cast<int32_t *>(lds + Npad * 32u);
    uint32_t *const sFlip = reinterpret_cast<uint32_t *>(lds + Npad * 36u);
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, r = lane & 31u, kg = lane >> 5, C0 = (uint32_t)a.C0, Wd = (uint32_t)a.Wd;
    const uint32_t pixels = (uint32_t)a.pixels, row_bytes = Wd * C0;  // (the host checks that the pixel count fits 31 bits)
    // Byte of the patch row and the row (0 .. 2) of this lane's slot j
    auto byte_of = [&](const uint32_t j) { return j < 9u ? j : (kg ? j - 2u : j - 9u); };
    auto row_of = [&](const uint32_t j) { return j < 9u ? 2u * kg : 1u; };
    uint32_t left[4] = {0u, 0u, 0u, 0u}, right[4] = {0u, 0u, 0u, 0u};  // slots in the column to the left, to the right
#pragma unroll
    for (uint32_t j = 0; j < 16; ++j) {
        const uint32_t b = byte_of(j);
        left[j >> 2] |= b < C0 ? 0xFFu << (8 * (j & 3u)) : 0u;
        right[j >> 2] |= b >= 2u * C0 ? 0xFFu << (8 * (j & 3u)) : 0u;
    }
    // Bytes of the tile's pixels: as loaded (a, b: eight and more bytes of either row), or, where a load could leave the image array, byte by
    // byte.  The loads of a wave's next tile are issued before it works on the current one, and those of its first before the tables.
    struct Bytes {
        uint32_t a[3], b[2];
    };
    auto inner = [&](const uint32_t tile) { return tile * 32u >= Wd + 1u && tile * 32u + 47u + Wd <= pixels; };
    auto position = [&](const uint32_t tile, uint32_t &p, uint32_t &x, uint32_t &y) {
        p = tile * 32u + r;
        p = p < pixels ? p : pixels - 1u;
        const uint32_t row = a.by_w.divide(p);
        x = p - row * Wd;
        y = row - a.by_h.divide(row) * (uint32_t)a.H;
    };
    auto gather = [&](const uint32_t tile, Bytes &got) {
        uint32_t p, x, y;
        if (inner(tile)) {
            p = tile * 32u + r;
            const uint8_t *const middle = a.x + ((uint64_t)p * C0 - C0);
            const uint8_t *const above = kg ? middle + row_bytes : middle - row_bytes;
            __builtin_memcpy(got.a, above, 12);
            __builtin_memcpy(got.b, middle + 7u * kg, 8);
        } else {
            position(tile, p, x, y);
            const uint32_t rows = (y > 0u ? 1u : 0u) | 2u | (y + 1u < (uint32_t)a.H ? 4u : 0u);
            const uint8_t *const centre = a.x + (uint64_t)p * C0;
            uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (uint32_t j = 0; j < 16; ++j) {
                const uint32_t b = byte_of(j), row = row_of(j);
                const bool in = b < 3u * C0 && ((rows >> row) & 1u) && (b >= C0 || x > 0u) && (b < 2u * C0 || x + 1u < Wd);
                const int64_t off = in ? ((int64_t)row - 1) * row_bytes + (int64_t)b - C0 : 0;
                const uint32_t v = centre[off];
                word[j >> 2] |= (in ? v : 0u) << (8 * (j & 3u));
            }
            got.a[0] = word[0], got.a[1] = word[1], got.b[0] = word[2], got.b[1] = word[3];
        }
    };
    auto operand = [&](const uint32_t tile, const Bytes &got) {
        uint32_t d[4] = {got.a[0], got.a[1], got.b[0], got.b[1]};
        if (inner(tile)) {
            uint32_t p, x, y;
            position(tile, p, x, y);
            const bool there = kg ? y + 1u < (uint32_t)a.H : y > 0u;
            const uint32_t row = there ? ~0u : 0u, l = x > 0u ? ~0u : 0u, rt = x + 1u < Wd ? ~0u : 0u;
            d[0] &= row, d[1] &= row;
            d[2] = __builtin_amdgcn_perm(got.b[0], got.a[2], 0x06050400u) & (row | 0xFFFFFF00u);
            d[3] = __builtin_amdgcn_alignbyte(got.b[1], got.b[0], 3u);
#pragma unroll
            for (int e = 0; e < 4; ++e) d[e] &= (l | ~left[e]) & (rt | ~right[e]);
        }
        v4i f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = (int)(d[e] ^ 0x80808080u);
        return f;
    };
    const uint32_t tiles = (pixels + 31u) / 32u, tile_step = blocks * (kFirstThreads / 64), first_tile = block * (kFirstThreads / 64) + wave;
    Bytes got = {};
    if (first_tile < tiles) gather(first_tile, got);
    // Per filter, by one thread: its nine words, threshold and flip flag are asked for together; then the filter as
    // bytes (-1 / +1, 0 in slots beyond the patch and beyond the last filter), and the sum of its weights (2 x set bits - patch
    // size) folded into the threshold.
    auto build_tables = [&](auto c0_tag) {
        constexpr int kC0 = decltype(c0_tag)::value;
        for (uint32_t n = t; n < Npad; n += kFirstThreads) {
            const bool there = n < (uint32_t)a.N;
            uint32_t w9[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) w9[i] = there ? a.W[(uint64_t)n * 9 + i] & ((1u << kC0) - 1u) : 0u;
            const int32_t tv = there ? a.T[n] : 0;
            const bool flipped = there && ((a.flip && a.flip[n]) != a.flip_all);
            uint32_t piece[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
            int32_t set = 0;
#pragma unroll
            for (int k = 0; k < 9 * kC0; ++k) {
                const int ky = k / (3 * kC0), b = k - 3 * kC0 * ky;
                const int slot = ky == 0 ? b : (ky == 2 ? 16 + b : (b < 7 ? 9 + b : 16 + 2 + b));
                const uint32_t bit = (w9[k / kC0] >> (k % kC0)) & 1u;
                piece[slot >> 2] |= (bit ? 0xFFu : 0x01u) << (8 * (slot & 3));
                set += (int32_t)bit;
            }
            uint4 *row = reinterpret_cast<uint4 *>(&sW[n * 32u]);
            row[0] = there ? make_uint4(piece[0], piece[1], piece[2], piece[3]) : make_uint4(0u, 0u, 0u, 0u);
            row[1] = there ? make_uint4(piece[4], piece[5], piece[6], piece[7]) : make_uint4(0u, 0u, 0u, 0u);
            const int32_t sum = there ? 2 * set - 9 * kC0 : 0;
            // |S + 128 sum| < 2^16: thresholds beyond +-2^30 decide the same way as +-2^30, and the difference cannot wrap
            const int32_t tc = tv < -(1 << 30) ? -(1 << 30) : (tv > (1 << 30) ? (1 << 30) : tv);
            sE[n] = tc - 1 - 128 * sum;
            const unsigned long long flips = __ballot(flipped);
            if ((lane & 31u) == 0u) sFlip[n / 32u] = (uint32_t)(flips >> lane);
        }
    };
    if (C0 == 3) {
        build_tables(std::integral_constant<int, 3>{});
    } else if (C0 == 2) {
        build_tables(std::integral_constant<int, 2>{});
    } else {
        build_tables(std::integral_constant<int, 1>{});
    }
    __syncthreads();
    // four output words (128 filters) at a time, so that a pixel's words leave as one 16-byte store: lanes of the
    // lower half write the bits, lanes of the upper half the ones plane
    const bool vec = a.ldo % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.out) | reinterpret_cast<uintptr_t>(a.ones)) & 15u) == 0;
    const uint32_t last_live = a.N % 32 ? (1u << (a.N % 32)) - 1u : ~0u;
    for (uint32_t tile = first_tile; tile < tiles; tile += tile_step) {
        const v4i af = operand(tile, got);
        const uint64_t p = (uint64_t)tile * 32u + r;
        const bool live = p < pixels;
        if (tiles - tile > tile_step) gather(tile + tile_step, got);
        for (uint32_t nb0 = 0; nb0 < Nw; nb0 += 4) {
            uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t nb = nb0 + u;
                if (nb >= Nw) break;
                const v4i wf = *reinterpret_cast<const v4i *>(&sW[(nb * 32u + r) * 32u + 16u * kg]);
                // acc[v]: what the sum for pixel r and filter 32 nb + 8 (v / 4) + 4 kg + v mod 4 lacks of its threshold, negative iff it meets it
                v16i acc;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4i e = *reinterpret_cast<const v4i *>(&sE[nb * 32u + 8u * q + 4u * kg]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[4 * q + i] = e[i];
                }
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf, af, acc, 0, 0, 0);
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // four sign bits, most significant first, one funnel shift each
                    uint32_t nib = 0;
#pragma unroll
                    for (int i = 3; i >= 0; --i) nib = __builtin_amdgcn_alignbit(nib, (uint32_t)acc[4 * q + i], 31);
                    bits |= nib << (8 * q);
                }
                word[u] = (or_halves(bits << (4u * kg)) ^ sFlip[nb]) & (nb == Nw - 1u ? last_live : ~0u);
            }
            if (!live) continue;
            uint32_t *dst = nullptr;
            if (kg == 0) {
                dst = a.out + p * a.ldo + nb0;
            } else if (a.ones) {
                dst = a.ones + p * a.ldo + nb0;
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) word[u] = nb0 + u == Nw - 1u ? last_live : ~0u;
            }
            if (dst) {
                if (vec && nb0 + 4 <= Nw) {
                    *reinterpret_cast<uint4 *>(dst) = make_uint4(word[0], word[1], word[2], word[3]);
                } else {
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u)
                        if (nb0 + u < Nw) dst[u] = word[u];
                }
            }
        }
    }
}

}  // namespace

bool conv_first_supports(int64_t C0, int64_t N, int KH, int KW, int pad, int stride) {
    return KH == 3 && KW == 3 && pad == 1 && stride == 1 && C0 >= 1 && C0 <= 3 && N >= 1 && N <= kFirstMaxN;
}

static int net_prep(const ConvPrepJobs &jobs, const FlagJobs &flags, NetPrep &p) {
    p.jobs = jobs, p.flags = flags;
    int64_t most = 0;
    for (int j = 0; j < flags.count; ++j) most = flags.n[j] > most ? flags.n[j] : most;
    const int64_t per_job = ceil_div(most, 256), flag_blocks = per_job * flags.count;
    int64_t blocks = 0;
    for (int j = 0; j < jobs.count; ++j) {
        p.jobs.first_block[j] = blocks;
        blocks += ceil_div(jobs.ld[j], 16);
    }
    p.jobs.first_block[jobs.count] = blocks;
    if (blocks + flag_blocks > 0x7FFF0000LL) return fail(QNN_ERR_SHAPE, "convnet: too many filters");
    p.flag_blocks = (uint32_t)flag_blocks, p.per_job = (uint32_t)(per_job > 0 ? per_job : 1), p.blocks = (uint32_t)(blocks + flag_blocks);
    return QNN_OK;
}

int launch_conv_class_thr(const ConvPrepJobs &jobs, const FlagJobs &flags, hipStream_t s) {
    NetPrep p;
    if (int rc = net_prep(jobs, flags, p)) return rc;
    if (p.blocks == 0) return QNN_OK;
    return QNN_LAUNCH("conv_class_thr", conv_class_thr_kernel, dim3(p.blocks), dim3(kFirstThreads), 0, s, p);
}

int launch_conv_first(const uint8_t *x, int64_t B, int H, int Wd, int C0, const uint32_t *W, int64_t N, const int32_t *T,
                      const uint8_t *flip, bool flip_all, uint32_t *out, uint32_t *ones, int64_t ldo, const ConvPrepJobs &jobs,
                      const FlagJobs &flags, hipStream_t s) {
    NetPrep p;
    if (int rc = net_prep(jobs, flags, p)) return rc;
    FirstConvArgs a;
    a.x = x, a.W = W, a.T = T, a.flip = flip, a.flip_all = flip_all, a.out = out, a.ones = ones, a.ldo = ldo;
    a.pixels = B * H * Wd, a.H = H, a.Wd = Wd, a.C0 = C0, a.N = (int)N;
    a.by_w = divider((uint32_t)Wd), a.by_h = divider((uint32_t)H);
    const int64_t tiles = ceil_div(a.pixels, 32);
    // a workgroup prepares the filter bytes once and then walks over pixel tiles: a few workgroups per compute unit (128 filters on 256 x 32 x 32
    // pixels: 512 workgroups 13.1 us, 768 12.3, 1024 13.0, 1536 14.6, 2048 15.0)
    const int64_t blocks = ceil_div(tiles, 4);
    const unsigned grid = (unsigned)(blocks < 768 ? blocks : 768);
    return QNN_LAUNCH("conv_first", conv_first_kernel, dim3(p.blocks + grid), dim3(kFirstThreads), first_lds(ceil_div(N, 32) * 32), s, a, p);
}

}  // namespace qnn
