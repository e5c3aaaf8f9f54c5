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
//   * Workgroup: four waves of 64 x 32 WBN on a tile of 128 x 64 WBN, and TWO workgroups on a compute unit: one multiplies while the other
//     stores its tile (14 % of the time at 8192^3 where one workgroup of four 128 x 128 waves had the unit to itself), runs its
//     threshold epilogue or waits at its barrier.
// Requirements (otherwise gemm_mfma_kernel takes the product): one plane per operand, rows of whole 64-byte groups
// starting on 16-byte boundaries, operands that span less than 4 GiB each.
#pragma once
#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"

namespace qnn {
namespace panel {

using mfma::v16f;
using mfma::v4i;

constexpr int kThreads = 256;
constexpr int WB = 2, BM = 128;   // blocks of 32 rows of a wave, rows of a tile
constexpr int kRowBytes = 64;     // bytes of a row per group: two steps of two 16-byte k-groups
constexpr int kGroupWords = kRowBytes / 4;

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int t) { return t == 0 ? v.x : (t == 1 ? v.y : (t == 2 ? v.z : v.w)); }

// kSign: threshold epilogue (Alg. 4: a^b = Sign(BatchNorm(a))) instead of int32 sums.
// WBN: 32-column blocks per wave along n, 4 (tile 128 x 256) or 2 (128 x 128).
template <bool kSign, int WBN>
__global__ __launch_bounds__(kThreads, 2) void gemm_panel_kernel(const GemmArgs g, const MfmaConst mc, uint32_t tiles_m,
                                                                  uint32_t tiles_n, uint32_t ngroups) {
    constexpr int WTN = 32 * WBN, BN = 2 * WTN;  // columns of a wave tile / of the workgroup tile
    constexpr uint32_t kPanelBytes = BM * kRowBytes, kGroupBytes = kPanelBytes + BN * kRowBytes;
    constexpr int kTable = 128;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kGroupBytes];
    __shared__ __attribute__((aligned(16))) uint32_t rw_table[4][kTable];
    __shared__ __attribute__((aligned(16))) int32_t thr_table[kSign ? 4 : 1][kSign ? kTable : 4];
    __shared__ __attribute__((aligned(16))) uint32_t flip_table[kSign ? 4 : 1][kSign ? kTable : 4];
    // int32 epilogue: per wave one 32 x 32 staging block, through which a block is turned from the accumulator layout
    // (a lane = one row) into whole 128-byte lines per row
    __shared__ __attribute__((aligned(16))) int32_t stage[kSign ? 1 : 4][kSign ? 4 : 32 * 32];
    static_assert(sizeof(lds) + sizeof(rw_table) + sizeof(thr_table) + sizeof(flip_table) + sizeof(stage) <= 80 * 1024, "two workgroups on a compute unit");

    const uint32_t lane = threadIdx.x & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1u;
    const uint32_t total_tiles = tiles_m * tiles_n;
    auto opaque = [](uint32_t x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    if constexpr (kSign) {  // flip flags default to "none" (complete long before the first epilogue reads them)
        flip_table[wave][lane] = 0u;
        flip_table[wave][lane + 64] = 0u;
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
    uint32_t off[kLoads];
    auto p_locate = [&](const uint32_t vb) __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(vb, total_tiles, tiles_m, tiles_n, tm, tn);
        const uint32_t ln = opaque(lane), row = 16u * wave + (ln >> 2), piece = ((ln & 3u) ^ (ln >> 4)) << 4;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const bool is_a = i < kLoadsA;
            const uint32_t last = (uint32_t)((is_a ? g.M : g.N) - 1);
            uint32_t at = (is_a ? tm * (uint32_t)BM + 64u * i : tn * (uint32_t)BN + 64u * (i - kLoadsA)) + row;
            at = at > last ? last : at;
            off[i] = at * ((uint32_t)(is_a ? g.A.ld : g.ldw) * 4u) + piece;
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
    auto load = [&](const int i, const uint32_t buf) __attribute__((always_inline)) {
        const uint8_t *const base = reinterpret_cast<const uint8_t *>(i < kLoadsA ? g.A.base : g.W) + p_G * (uint32_t)kRowBytes;
        const uint32_t dst = lds_base + buf + (uint32_t)i * 4096u + wave * 1024u;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off[i]), "s"(base) : "memory");
    };
    // the next group has landed and this wave's LDS reads have returned
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // (the second group may still be on its way)
    auto first_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kLoads) : "memory"); };

    p_locate(vb0);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load(i, 0u);
    p_advance();
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
            rw[i] += (int32_t)__builtin_popcount(word_of(c.W[i], t));
            asm("" : "+v"(rw[i]));
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

    Step cur, nxt;
    fetch(0, rd, cur);
    uint32_t vb = vb0;
    for (uint32_t done = 0; done < n_mine; ++done, vb += gridDim.x) {
        uint32_t tile_m, tile_n;
        tile_of_block(vb, total_tiles, tiles_m, tiles_n, tile_m, tile_n);
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
        if constexpr (kSign) load_thresholds_to_lds<WBN>(g, n_wave, thr_table[wave], flip_table[wave]);
        for (uint32_t G = 0; G < ngroups; ++G) {
            const uint32_t other = kGroupBytes - rd;
            p_advance();
            fetch(1, rd, nxt);
            __builtin_amdgcn_sched_barrier(0);
            phase(p0, cur, nothing);
            phase(p1, cur, nothing);
            phase(p2, cur, nothing);
            phase(p3, cur, nothing);
            barrier();  // every wave holds the second step's words: the buffer is free
            fetch(0, other, cur);
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
        wave_finish<kSign, WBN, kLoads>(g, mc, acc, ra, rw, rw_table[wave], thr_table[wave], flip_table[wave], stage[kSign ? 0 : wave], m_wave, n_wave);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads beyond the last tile)
}

typedef void (*KernelFn)(const GemmArgs, const MfmaConst, uint32_t, uint32_t, uint32_t);
// narrow: the 128 x 128 workgroup tile
KernelFn find_kernel(bool sign, bool narrow);
KernelFn wide_kernel();  // int32 sums, 256 x 256 tiles, rows of whole 128-byte groups (qnn_gemm_panel_wide_kernel.h)
constexpr int kWideGroupWords = 32;

}  // namespace panel
}  // namespace qnn
