// Matrix-core engine, uint8 left operand against +-1 weights kept as bits, threshold output: the first layer of Alg. 4 on 8-bit inputs
// (by Eq. (FirstLayer) the eight weighted plane products are x . w on the codes themselves).
//
// 16 consecutive codes of a row, minus 128, are an int8 operand of v_mfma_i32_32x32x32_i8 as they stand.  The weights go through memory and
// LDS as bits and become operands of +-64 in registers, with two instructions per register: a shift and (x & 0x80..) | 0x40...  For that
// their bits are put in the order of the operands once per call (weight_image_kernel).  The sums are 64 times
//   sum_k (x[m][k] - 128) w[n][k],  and C[m][n] is that plus 128 sum_k w[n][k],
// a term per weight row that the image kernel writes as well.  Pieces of 16 elements beyond K read as zeros, i.e. -128, and meet as many
// weights of +64 as of -64.
//   The sums start from -64 (T - term), so that a finished sum's sign is its bit and the epilogue is one instruction per element; with the
// comparison at the end (shift, scale, two terms, difference, sign) that was six, a quarter of the instructions of a tile of 784 codes:
// 10000 x 784 -> 4096 38.5 -> 34.3 us.
// Workgroup: four waves of 64 x 32 NB on a tile of 128 x 64 NB, two on a compute unit (they cover each other's barriers and thresholds); both
// operands of a group of 128 elements of k come in straight to LDS, two group buffers.
// Bound: the card's power.  8192 x 4096 x 4096 takes 116 us with 56 % of the cycles in matrix instructions on random codes, 88 on constant
// ones; multiplying what LDS holds as it is, without the unpacking, took 109.  Before, with the weights as bytes and one workgroup of
// 256 x 256 tiles on a unit (or, for fewer rows than the weights' bytes leave room for in the workspace, bits expanded by every wave;
// whole forward step with a 10-neuron second layer): 10000 x 784 -> 4096 59 -> 51 us, 4096 x 784 -> 4096 34.5 -> 26, 2000 x 784 -> 4096 28 ->
// 19.7, 10000 x 4096 -> 4096 174 -> 155, 3000 x 3072 -> 1000 33 -> 28.
#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"

namespace qnn {
namespace codes {

namespace {

using mfma::v16i;
using mfma::v4i;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256, kGroupK = 128, kMB = 2, kBM = 128;
constexpr uint32_t kBlockRows = 128, kBlockBytes = kBlockRows * kGroupK / 8;  // of the weights' image
constexpr uint32_t kPanel = kBM * kGroupK, kGroup = kPanel + 2 * kBlockBytes;

struct CodesArgs {
    uint32_t a_bytes;  // size of the codes
    uint32_t image_blocks;
    uint32_t halves;   // of groups, ceil(K / 64)
    Tiles tiles;
};

template <int NB>
__global__ __launch_bounds__(kThreads, 2) void gemm_codes_kernel(const GemmArgs g, const CodesArgs x) {
    constexpr uint32_t kTable = 32 * NB, kLoadsA = kPanel / 4096, kLoads = kLoadsA + 1;  // of 1024 bytes each, per wave
    // two group buffers; per wave the thresholds, flip flags and weight rows' terms of its columns as they arrive, and what its sums start from
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kGroup + 4 * 4 * kTable * 4];
    static_assert(sizeof(lds) <= 80 * 1024, "two workgroups on a compute unit");
    const uint32_t lane = threadIdx.x & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1u;
    const uint32_t total = x.tiles.total, groups = (x.halves + 1u) / 2u, K = (uint32_t)g.K;
    const uint32_t lds_base = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds);
    uint32_t *const rw_tab = reinterpret_cast<uint32_t *>(lds + 2 * kGroup) + wave * 4u * kTable;
    int32_t *const thr_tab = reinterpret_cast<int32_t *>(rw_tab + kTable);
    uint32_t *const flip_tab = rw_tab + 2 * kTable;
    int32_t *const start_tab = thr_tab + 2 * kTable;
#pragma unroll
    for (uint32_t h = 0; h < kTable; h += 64) flip_tab[h + lane] = 0u;  // flip flags default to "none"
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (before the loads that write the same words)
    auto opaque = [](uint32_t v) __attribute__((always_inline)) {  // keeps address arithmetic where it is used
        asm volatile("" : "+v"(v));
        return v;
    };

    // The producer's cursor (a tile, group p_G) runs two groups ahead of the multiplication.  A load of codes covers 8 rows x 128 bytes: lane
    // i lands in piece i mod 8 of row i / 8 and fetches piece (i mod 8) xor (row / 2 mod 8), which spreads LDS reads over the banks.
    const uint32_t vb0 = blockIdx.x, n_mine = (total - vb0 + gridDim.x - 1u) / gridDim.x;
    uint32_t p_G = 0, p_item = 0, p_in = 0, off[kLoadsA];  // p_in: of this lane's piece in its row
    const uint8_t *p_w;
    auto p_locate = [&](const uint32_t vb) __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(vb, x.tiles, tm, tn);
        const uint32_t last = (uint32_t)(g.M - 1), row = 8u * wave + (opaque(lane) >> 3);
#pragma unroll
        for (uint32_t i = 0; i < kLoadsA; ++i) {
            uint32_t at = tm * (uint32_t)kBM + 32u * i + row;
            at = at > last ? last : at;
            off[i] = at * (uint32_t)g.A.ld;
        }
        p_w = reinterpret_cast<const uint8_t *>(g.w_image) + (uint64_t)(tn * (uint32_t)NB / 2u) * kBlockBytes + wave * 1024u;
    };
    auto p_piece = [&]() __attribute__((always_inline)) {
        const uint32_t ln = opaque(lane);
        p_in = p_G * (uint32_t)kGroupK + (((ln & 7u) ^ ((ln >> 4) | ((wave & 1u) << 2))) << 4);
    };
    auto p_advance = [&]() __attribute__((always_inline)) {
        p_w += (uint64_t)x.image_blocks * kBlockBytes;
        if (++p_G == groups) {
            asm volatile("" ::: "memory");  // keeps the branch a branch
            p_G = 0;
            ++p_item;
            // (after the last tile the loads start over and are never used)
            p_locate(p_item < n_mine ? vb0 + p_item * gridDim.x : vb0);
        }
        p_piece();
    };
    const uint64_t a_base = reinterpret_cast<uint64_t>(g.A.base);
    const u32x4 a_rsrc = {(uint32_t)a_base, (uint32_t)(a_base >> 32) & 0xFFFFu, x.a_bytes, 0x00027000u};
    const uint32_t lane16 = lane * 16u;
    auto load = [&](const uint32_t i, const uint32_t buf) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + buf + i * 4096u + wave * 1024u;
        if (i < kLoadsA) {
            const uint32_t voff = p_in < K ? off[i % kLoadsA] + p_in : 0xFFFFFFF0u;  // (beyond K: zeros)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(dst), "v"(voff), "s"(a_rsrc) : "memory");
        } else {
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(lane16), "s"(p_w) : "memory");
        }
    };
    // the next group has landed and this wave's LDS reads have returned
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // thresholds, flip flags and weight rows' terms of a tile on their way to the wave's tables
    auto load_columns = [&](const uint32_t vb) __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(vb, x.tiles, tm, tn);
        const int64_t n0 = (int64_t)tn * (64 * NB) + wn * (32 * NB);
        panel::load_thresholds_to_lds<NB>(g, n0, thr_tab, flip_tab);
        const uint32_t rw_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t *)rw_tab);
#pragma unroll
        for (uint32_t h = 0; h < kTable; h += 64) {
            int64_t n = n0 + h + opaque(lane);
            if (n > g.N - 1) n = g.N - 1;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(rw_lds + 4u * h), "v"((uint32_t)n * 4u), "s"(g.rw_scaled) : "memory");
        }
    };

    load_columns(vb0);
    p_locate(vb0);
    p_piece();
#pragma unroll
    for (uint32_t i = 0; i < kLoads; ++i) load(i, 0u);
    p_advance();
#pragma unroll
    for (uint32_t i = 0; i < kLoads; ++i) load(i, kGroup);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kLoads) : "memory");
    uint32_t rd = 0u;  // byte offset of the group buffer being consumed

    struct Half {  // 64 elements of k, two steps; lane (r, kg) holds the 16 elements 16 kg .. of a step of its rows
        v4i a[2][kMB];
        uint32_t w[NB];
    };
    auto fetch = [&](const uint32_t h, const uint32_t buf, Half &f) __attribute__((always_inline)) {
        const uint32_t piece = (kg ^ ((r >> 1) & 7u)) << 4;
        const uint8_t *const pa = lds + (buf + (wm * (32u * kMB) + r) * (uint32_t)kGroupK);
#pragma unroll
        for (uint32_t t = 0; t < 2; ++t)
#pragma unroll
            for (int b = 0; b < kMB; ++b) f.a[t][b] = *reinterpret_cast<const v4i *>(pa + (piece ^ (64u * h + 32u * t)) + b * (32 * kGroupK));
        const uint32_t *const pw = reinterpret_cast<const uint32_t *>(lds + (buf + kPanel)) + (NB == 4 ? wn * (kBlockBytes / 4) : wn * 64u) + (2u * h + kg) * kBlockRows + r;
#pragma unroll
        for (int b = 0; b < NB; ++b) f.w[b] = pw[32 * b];
    };
    v16i acc[NB][kMB];  // [n block][m block]
    // in registers: with literals in their place the compiler takes an instruction more
    uint32_t top = 0x80808080u, next = 0x40404040u;
    asm volatile("" : "+v"(top), "+s"(next));
    auto multiply = [&](const Half &f, const int t, auto between) __attribute__((always_inline)) {
        v4i a[kMB];
#pragma unroll
        for (int j = 0; j < kMB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) a[j][e] = f.a[t][j][e] ^ (int)0x80808080u;  // the codes minus 128
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            v4i w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (int)(((f.w[i] << (7 - 4 * t - e)) & top) | next);
#pragma unroll
            for (int j = 0; j < kMB; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, a[j], acc[i][j], 0, 0, 0);
            between((uint32_t)i);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto nothing = [](uint32_t) __attribute__((always_inline)) {};

    Half cur, nxt;
    fetch(0, rd, cur);
    uint32_t vb = vb0;
    for (uint32_t done = 0; done < n_mine; ++done, vb += gridDim.x) {
        uint32_t tile_m, tile_n;
        tile_of_block(vb, x.tiles, tile_m, tile_n);
        const int64_t m_wave = (int64_t)tile_m * kBM + wm * (32 * kMB), n_wave = (int64_t)tile_n * (64 * NB) + wn * (32 * NB);
        // What has arrived (before a barrier): the sums start from -64 (T - term), so that a sum's sign is its bit.  |s| < 2^24, so a
        // difference clamped there decides the same, and 64 (s - difference) stays within 32 bits.
        uint32_t flips[NB];
#pragma unroll
        for (uint32_t h = 0; h < kTable / 64; ++h) {
            const uint32_t at = 64u * h + opaque(lane);
            constexpr int32_t kMost = 1 << 24, kMostT = 1 << 26;
            const int32_t t = thr_tab[at];
            int32_t d = (t < -kMostT ? -kMostT : (t > kMostT ? kMostT : t)) - (int32_t)rw_tab[at];
            d = d < -kMost ? -kMost : (d > kMost ? kMost : d);
            start_tab[at] = -64 * d;
            const uint64_t flip = __ballot(flip_tab[at] == 0u);
            flips[2 * h] = (uint32_t)flip, flips[2 * h + 1] = (uint32_t)(flip >> 32);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the wave's own LDS operations are done
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int32_t *const start_of = start_tab + 32 * i + 4u * (opaque(lane) >> 5);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i start = *reinterpret_cast<const v4i *>(start_of + 8 * q);
#pragma unroll
                for (int j = 0; j < kMB; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] = start[e];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (done + 1u < n_mine) load_columns(vb + gridDim.x);
        uint32_t G = 0;
        do {  // (a loop that might not run would hold the sums' start and the sums in registers of their own)
            const uint32_t other = kGroup - rd;
            p_advance();
            fetch(1, rd, nxt);
            __builtin_amdgcn_sched_barrier(0);
            multiply(cur, 0, nothing);
            multiply(cur, 1, nothing);
            barrier();  // every wave holds the second half's operands: the buffer is free
            fetch(0, other, cur);
            if (2u * G + 1u == x.halves) {  // (nothing in the group's second half)
#pragma unroll
                for (uint32_t i = 0; i < kLoads; ++i) load(i, rd);
                rd = other;
                break;
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(nxt, 0, [&](const uint32_t i) __attribute__((always_inline)) {
                constexpr uint32_t kEach = (kLoads + NB - 1) / NB;
#pragma unroll
                for (uint32_t p = 0; p < kEach; ++p)
                    if (kEach * i + p < kLoads) load(kEach * i + p, rd);
            });
            multiply(nxt, 1, nothing);
            rd = other;
        } while (++G < groups);
        // The sums are pinned here: otherwise the compiler moves matrix-core instructions down into the epilogue
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < kMB; ++j) asm volatile("" : "+v"(acc[i][j]));
        uint32_t word[NB];
        const uint32_t kg_here = opaque(lane) >> 5;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            uint32_t both[kMB];
#pragma unroll
            for (int j = 0; j < kMB; ++j) {
                uint32_t bits = 0;  // register 4 q + e: column 8 q + 4 kg + e of the block's 32
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t nib = 0;
#pragma unroll
                    for (int e = 3; e >= 0; --e) nib = __builtin_amdgcn_alignbit(nib, (uint32_t)acc[i][j][4 * q + e], 31);
                    bits |= nib << (8 * q);
                }
                both[j] = mfma::or_halves(bits << (4u * kg_here));
            }
            word[i] = (kg_here ? both[1] : both[0]) ^ flips[i];
            __builtin_amdgcn_sched_barrier(0);
        }
        panel::store_words<NB>(g, word, m_wave + opaque(lane), n_wave);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads beyond the last tile)
}

// The weights' image: [group of 128 elements][block of 128 rows][half of 64][kg][row], a word each: its bit 8 j + 4 t + d stands for element
// 64 half + 32 t + 16 kg + 4 d + j, clear where the weight is +1.  Pieces of 16 elements beyond K alternate.  rw_scaled[n] = 128 sum_k
// w[n][k].  A thread takes one of a group's four words, a workgroup 16 rows, its waves the groups in turn.  Rows beyond N are not written
// (their columns of C do not exist).
__global__ __launch_bounds__(256) void weight_image_kernel(const uint32_t *__restrict__ W, uint32_t N, uint32_t K, int64_t ldw, uint32_t groups,
                                                           uint32_t image_blocks, uint32_t *__restrict__ image, int32_t *__restrict__ rw_scaled) {
    __shared__ int32_t counts[4][64];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, half = (lane >> 4) >> 1, kg = (lane >> 4) & 1u, n = blockIdx.x * 16u + (lane & 15u);
    int32_t pop = 0;
    if (n < N) {
        for (uint32_t G = wave; G < groups; G += 4) {
            uint32_t o = 0;
#pragma unroll
            for (uint32_t t = 0; t < 2; ++t) {
                const uint32_t word = 4u * G + 2u * half + t;
                if (32u * word + 16u * kg < K) {
                    const uint32_t bits = (W[n * ldw + word] >> (16u * kg)) & 0xFFFFu;
                    pop += __builtin_popcount(bits);
#pragma unroll
                    for (uint32_t d = 0; d < 4; ++d) o |= ((((~bits >> (4u * d)) & 0xFu) * 0x00204081u) & 0x01010101u) << (4u * t + d);
                } else {
                    o |= 0x05050505u << (4u * t);
                }
            }
            image[((uint64_t)G * image_blocks + n / kBlockRows) * (kBlockBytes / 4) + (2u * half + kg) * kBlockRows + n % kBlockRows] = o;
        }
    }
    counts[wave][lane] = pop;
    __syncthreads();
    if (threadIdx.x < 16 && n < N) {
        pop = 0;
        for (int q = 0; q < 16; ++q) pop += counts[q >> 2][16 * (q & 3) + lane];
        rw_scaled[n] = 256 * pop - 128 * (int32_t)K;
    }
}

// The same product for few rows, straight from the weights' bits: tiles of 32 x 32 whose waves share k, 32 elements at a time.  Bound: latency, so all
// loads of a wave that fit its registers are on their way together, the sums meet once in LDS, and no launch prepares anything (bit planes and their
// product took two launches and four products of digits).  A word's half of 16 bits becomes 0 / 1 bytes, four with one multiplication:
// with y = x - 128, sum x w = 2 sum y b - sum y + 128 (2 pop - K).
template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void gemm_codes_small_kernel(const GemmArgs g, const Tiles tiles) {
    constexpr uint32_t kAhead = kWaves == 16 ? 2 : 4;  // units of 32 elements whose loads are on their way together
    __shared__ __attribute__((aligned(16))) int32_t part[kWaves][32][36];
    __shared__ int32_t part_a[kWaves][32], part_w[kWaves][32];
    const uint32_t lane = threadIdx.x & 63u, r = lane & 31u, kg = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t tm, tn;
    tile_of_block(blockIdx.x, tiles, tm, tn);
    const uint32_t M = (uint32_t)g.M, N = (uint32_t)g.N, K = (uint32_t)g.K, m0 = 32u * tm, n0 = 32u * tn, units = (K + 31u) / 32u;
    // (rows beyond the last repeat it and are not stored)
    const uint8_t *const codes = reinterpret_cast<const uint8_t *>(g.A.base) + (uint64_t)(m0 + r < M ? m0 + r : M - 1u) * (uint64_t)g.A.ld;
    const uint32_t n = n0 + r < N ? n0 + r : N - 1u;
    const uint32_t *const weights = g.W + (uint64_t)n * (uint64_t)g.ldw;
    const int32_t T = g.epi.T[n];
    const uint32_t flip = g.epi.flip ? g.epi.flip[n] : 0u;
    v16i acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0;
    int32_t sum = 0, pop = 0;
    for (uint32_t u0 = wave; u0 < units; u0 += kWaves * kAhead) {
        v4i a[kAhead];
        uint32_t word[kAhead];
        bool in[kAhead];
#pragma unroll
        for (uint32_t i = 0; i < kAhead; ++i) {
            const uint32_t u = u0 + kWaves * i, k = 32u * u + 16u * kg;
            in[i] = k < K;  // (K is a multiple of 16)
            a[i] = *reinterpret_cast<const v4i *>(codes + (in[i] ? k : 0u));
            word[i] = weights[u < units ? u : 0u];
        }
#pragma unroll
        for (uint32_t i = 0; i < kAhead; ++i) {
            const uint32_t bits = in[i] ? (word[i] >> (16u * kg)) & 0xFFFFu : 0u;
            v4i w;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[i][e] = in[i] ? a[i][e] ^ (int)0x80808080u : 0;
                sum = __builtin_amdgcn_sdot4(a[i][e], 0x01010101, sum, false);
                w[e] = (int)(__umul24((bits >> (4 * e)) & 0xFu, 0x00204081u) & 0x01010101u);
            }
            pop += __builtin_popcount(bits);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, a[i], acc, 0, 0, 0);
        }
    }
    // register 4 q + e: row r of the tile, column 8 q + 4 kg + e
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<v4i *>(&part[wave][r][8 * q + 4 * kg]) = v4i{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    sum = mfma::sum_halves(sum), pop = mfma::sum_halves(pop);
    if (kg == 0) part_a[wave][r] = sum, part_w[wave][r] = pop;
    __syncthreads();
    // a lane keeps its column, a ballot packs two rows
    const bool live = n0 + r < N;
    for (uint32_t row0 = 2u * wave; row0 < 32u; row0 += 2u * kWaves) {
        const uint32_t row = row0 + kg;
        int32_t s = 0, sa = 0, sw = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += part[w][row][r], sa += part_a[w][row], sw += part_w[w][r];
        const int32_t value = 2 * s - sa + 128 * (2 * sw - (int32_t)K);
        const uint64_t bits = __ballot(live && ((value >= T) != (flip != 0u)));
        if (r == 0u && m0 + row < M) g.epi.out_bits[(int64_t)(m0 + row) * g.epi.ldo + tn] = (uint32_t)(bits >> lane);
    }
}

// (a tile of 128 columns brings in the block beyond its own too)
int64_t blocks_of(int64_t N) { return ceil_div(N, kBlockRows) + 1; }

}  // namespace

size_t image_bytes(int64_t N, int64_t K) { return (size_t)(ceil_div(K, kGroupK) * blocks_of(N)) * kBlockBytes; }

bool supports(const GemmArgs &g) {
    // (the sums are below 64 x 128 K; offsets into the codes are 32-bit)
    return g.A.rows_are_bytes && g.w_image && g.rw_scaled && g.epi.T && g.K < 131072 && (long double)g.M * g.A.ld < 4294967296.0L && g.N < 0x7FFFFFF0;
}

// Forward step with a 10-neuron second layer, us, otherwise / this.
//   No room for the image, so that bits would be expanded per wave by tiles of 256 x 256: up to 3840 tiles of up to 1024 codes, 2816 of more, whatever the
//   rows (784 codes: 300 rows, 4096 neurons 37.3 / 23.4, 500 rows, 7400 neurons 28.8 / 24.1, beyond it 500 rows, 32768 neurons 40.5 / 80.7; 3072 codes: 500
//   rows, 5376 neurons 78 / 65, 7392 neurons 79 / 87; 8192 codes, 1000 rows, 65536 neurons 746 / 3565).
//   Bit planes otherwise: sums beyond 2^24, for which only the VALU is left, always (65536 codes, 512 neurons, 200 rows 2530 / 122).  Otherwise up
//   to 8192 codes and 49152 steps of 32 codes (784 codes, 512 neurons: 32 rows 14.0 / 10.6, 3000 rows 27.3 / 19.1; 3072 codes, 512 neurons, 1000 rows
//   22.9 / 17.4; beyond that 4096 neurons, 200 rows 27.0 / 28.7; 12288 codes, 512 neurons, 32 rows 26.6 / 27.1, 2000 rows 73 / 91), and of up to 256 codes
//   in rows of whole 128-byte lines up to 20480 (128 codes: 600 rows, 6720 neurons 21.3 / 19.4, 10944 neurons 22.5 / 27.0, but 112 codes 22.5 / 20.2, and 27.6 in
//   rows of 128; 256 codes: 100 rows, 8192 neurons 15.6 / 12.2, 32768 neurons 25.9 / 29.6).
bool small_preferred(const GemmArgs &g, bool large, bool has_image) {
    if (large && has_image) return false;
    if (!(g.A.rows_are_bytes && g.epi.T && g.K < 131072 && g.K % 16 == 0 && g.A.ld % 16 == 0 && reinterpret_cast<uintptr_t>(g.A.base) % 16 == 0 &&
          g.pw.mode == QNN_PLANE_SIGN && g.pw.count == 1 && g.pw.coef[0] == 1 && g.M < 0x7FFFFFE0 && g.N < 0x7FFFFFE0))
        return false;
    const int64_t tiles = ceil_div(g.M, 32) * ceil_div(g.N, 32), steps = ceil_div(g.K, 32);
    if (tiles >= 1 << 24) return false;
    if (large) return tiles <= (steps <= 32 ? 3840 : 2816);
    if (255 * g.K > 1 << 24) return true;
    return steps <= 256 && tiles * steps <= (steps <= 8 && g.A.ld % 128 == 0 ? 20480 : 49152);
}

int launch_small(const GemmArgs &g, hipStream_t s) {
    const int64_t m = ceil_div(g.M, 32), n = ceil_div(g.N, 32);
    const bool many = m * n > 512;
    return QNN_LAUNCH("gemm_codes_small", (many ? gemm_codes_small_kernel<4> : gemm_codes_small_kernel<16>), dim3((unsigned)(m * n)), dim3(many ? 256 : 1024), 0, s, g,
                      make_tiles(m, n));
}

int launch_weight_image(const GemmArgs &g, hipStream_t s) {
    return QNN_LAUNCH("weight_image", weight_image_kernel, dim3((unsigned)ceil_div(g.N, 16)), dim3(256), 0, s, g.W, (uint32_t)g.N, (uint32_t)g.K, g.ldw,
                      (uint32_t)ceil_div(g.K, kGroupK), (uint32_t)blocks_of(g.N), const_cast<uint32_t *>(g.w_image), const_cast<int32_t *>(g.rw_scaled));
}

int launch(const GemmArgs &g, hipStream_t s) {
    const int64_t cus = compute_units(), tiles_m = ceil_div(g.M, kBM);
    // 128 x 256 or 128 x 128 by the time of their rounds, with two workgroups and with one on a unit (whole forward step with a 10-neuron
    // second layer, us, 128 x 256 / 128 x 128: 10000 x 784 -> 4096 51 / 60, -> 2048 31.0 / 31.6, -> 1000 23.6 / 22.8, 3000 x 3072 -> 1000 34 / 28;
    // three workgroups of 128 x 128 tiles: 56, 31.2, 22.3, 28)
    auto rounds = [cus](int64_t tiles, double two, double one) {
        const int64_t rest = tiles % (2 * cus);
        return (double)(tiles / (2 * cus)) * two + (rest == 0 ? 0.0 : (rest <= cus ? one : two));
    };
    const int64_t wide = tiles_m * ceil_div(g.N, 256), narrow = tiles_m * ceil_div(g.N, 128);
    const bool is_wide = rounds(wide, 2.0, 1.3) <= rounds(narrow, 1.22, 0.95);
    const int64_t total = is_wide ? wide : narrow;
    if (total > 0x7FFFFFFF) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
    CodesArgs x;
    x.a_bytes = (uint32_t)((g.M - 1) * g.A.ld + g.K), x.image_blocks = (uint32_t)blocks_of(g.N), x.halves = (uint32_t)ceil_div(g.K, 64);
    x.tiles = make_tiles(tiles_m, total / tiles_m);
    return QNN_LAUNCH("gemm_codes", (is_wide ? gemm_codes_kernel<4> : gemm_codes_kernel<2>), dim3((unsigned)(total < 2 * cus ? total : 2 * cus)),
                      dim3(kThreads), 0, s, g, x);
}

}  // namespace codes
}  // namespace qnn
