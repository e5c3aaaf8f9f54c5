// Matrix-core engine, panel-fed kernel for two operands of int8 values: bit planes merged to one byte per element by
// merge_planes_kernel (Sec. 2.6 / Sec. 3: the weighted sum of the plane products is the product of the values the planes stand for),
// with int32 sums as output and no correction terms.
//
// With both operands as bytes the main loop is loads to LDS, LDS reads and the matrix-core instructions (v_mfma_i32_32x32x32_i8).
// As in gemm_panel_wide_kernel the operands come in through LDS: the rows the workgroup shares are loaded as whole 128-byte
// lines straight to LDS (global_load_lds), a group of 128 elements of k (four steps of 32) at a time into two group
// buffers; 16-byte piece c of row r sits at piece c xor (r / 2 mod 8), which puts the 16 rows that a ds_read_b128 serves at a time
// on 16 different quarters of the banks (with r mod 8 rows r and r + 8 met: half of the LDS cycles were conflicts).
// Workgroup tile 256 x 256 on eight waves of 128 x 64, two per SIMD: a load to LDS holds the issuing wave for tens of cycles and
// every group ends in a barrier; with one wave of 128 x 128 per SIMD (the earlier shape of this kernel) the matrix cores waited
// with it.  A group takes 2600 cycles of which 2048 are matrix-core time (1.08 us on zeros; random operands, under whose switching the
// card lowers its clock from 2.4 to about 2.1 GHz, 1.30 us).  Where rounds of such tiles leave much of the chip idle, tiles have 192 or
// 128 rows (see bytes_tiles).
#pragma once
#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"

namespace qnn {
namespace bytes_panel {

using mfma::MfmaConst;
using mfma::v16i;
using mfma::v4i;

constexpr int kThreads = 512;
constexpr int BM = 256, BN = 256;  // the largest tile: a wave's part of it is 128 rows x 64 columns
constexpr int kRowBytes = 128;                         // codes of a row per group
constexpr int kPanelBytes = BM * kRowBytes;            // one operand's rows of a group
constexpr int kGroupBytes = 2 * kPanelBytes;
constexpr int kGroupK = 128;

// kTail (grid = a multiple of 16 workgroups, fewer than there are tiles, and at most half a grid of tiles in the last round): that
// round's tiles are taken as halves of 128 columns by two workgroups each.
// WB: blocks of 32 rows per wave, so the tile has 64 WB rows: 256, 192 or 128 (see bytes_tiles).
template <bool kTail, int WB>
__global__ __launch_bounds__(kThreads, 2) void gemm_bytes_panel_kernel(const GemmArgs g, const MfmaConst mc, uint32_t tiles_m,
                                                                       uint32_t tiles_n, uint32_t ngroups) {
    constexpr int kLoadsPerGroup = WB + 4;  // loads to LDS that a wave issues per group
    static_assert(!kTail || WB == 4, "halves of whole tiles");
    // One LDS array: two group buffers, then the per-wave 32 x 32 staging blocks of the epilogue (all 160 KiB).
    constexpr int kRingBytes = 2 * kGroupBytes;
    constexpr int kStageBytes = 32 * 32 * 4, kTailBytes = (kThreads / 64) * kStageBytes;
    static_assert(kRingBytes + kTailBytes <= 160 * 1024, "LDS of a compute unit");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kRingBytes + kTailBytes];
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const uint32_t total_tiles = tiles_m * tiles_n;
    const uint32_t K = (uint32_t)g.K;
    int32_t *const stage_w = reinterpret_cast<int32_t *>(lds + kRingBytes + wave * kStageBytes);

    // lane-dependent values are re-derived behind an opaque copy wherever they are used (address arithmetic that the
    // compiler computes once before the loops ends up spilled, and a reload in the main loop stalls the wave)
    auto opaque = [](uint32_t x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    const uint32_t tid = (uint32_t)t;
    const uint32_t lds_base = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds);

    // ------------------------------------------------------------------------------------------------ producer
    // The producer's cursor (tile p_vb, group p_G) runs two groups ahead of the multiplication.  Everything that depends on
    // the tile only is worked out when the cursor enters a tile.  This workgroup's tiles: vb0, vb0 + gridDim.x, ... (n_mine of
    // them); kTail: the tiles of the whole rounds, then half of a tile of the last round, shared with a workgroup of the same XCD.
    const uint32_t vb0 = blockIdx.x;
    const uint32_t whole_rounds = total_tiles / gridDim.x;
    const uint32_t n_mine = kTail ? whole_rounds : (total_tiles - vb0 + gridDim.x - 1u) / gridDim.x;
    const uint32_t tail_vb = whole_rounds * gridDim.x + ((vb0 >> 4) << 3) + (vb0 & 7u);
    const bool has_half = kTail && tail_vb < total_tiles;
    const uint32_t half_col = ((vb0 >> 3) & 1u) * (uint32_t)(BN / 2);
    uint32_t p_vb = vb0, p_G = 0, p_item = 0;
    uint32_t a_off[WB], w_off[4];  // byte offsets of the rows this lane loads (weights: plus its piece of the line)
    uint32_t p_jb = 0;            // byte offset within an activation row of this lane's piece of the group at the cursor
    const uint32_t lda_bytes = (uint32_t)g.A.ld, ldw_bytes = (uint32_t)g.ld_w_bytes;
    const uint32_t last_m = (uint32_t)(g.M - 1), last_n = (uint32_t)(g.N - 1);
    // a load covers 8 rows x 128 bytes: lane i lands in slot i mod 8 of row i / 8 and therefore fetches piece
    // (i mod 8) xor (row / 2 mod 8); load i of a panel takes rows 64 i + 8 wave .. + 7
    auto p_locate = [&]() __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(p_vb, total_tiles, tiles_m, tiles_n, tm, tn);
        const uint32_t tt = opaque(tid);
        const uint32_t pr = tt >> 3, piece = (tt & 7u) ^ ((tt >> 4) & 7u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < WB) {
                uint32_t m = tm * (uint32_t)(64 * WB) + (uint32_t)(64 * i) + pr;
                m = m > last_m ? last_m : m;
                a_off[i] = m * lda_bytes;
            }
            uint32_t n = tn * (uint32_t)BN + (uint32_t)(64 * i) + pr;
            n = n > last_n ? last_n : n;
            w_off[i] = n * ldw_bytes + piece * 16u;
        }
    };
    auto p_piece = [&]() __attribute__((always_inline)) {
        const uint32_t tt = opaque(tid);
        const uint32_t jb = p_G * (uint32_t)kGroupK + (((tt & 7u) ^ ((tt >> 4) & 7u)) << 4);
        p_jb = jb < K ? jb : 0u;  // a piece beyond the row reads the row's first bytes (valid memory, meets zero weights)
    };
    auto p_advance = [&]() __attribute__((always_inline)) {
        ++p_G;
        if (p_G == ngroups) {
            asm volatile("" ::: "memory");  // keeps the branch a branch
            p_G = 0;
            ++p_item;
            if (p_item < n_mine)
                p_vb = vb0 + p_item * gridDim.x;
            else if (has_half && p_item == n_mine)
                p_vb = tail_vb;
            // (after the last tile the loads are repeated and never used)
            p_locate();
        }
        p_piece();
    };
    // 16 bytes per lane from base + voff + vadd to LDS address lds_addr + 16 * lane.  The address travels in M0; the
    // addition sits between the write of M0 and the load, where an instruction has to be anyway.
    auto load16_to_lds = [](const void *base, uint32_t voff, uint32_t vadd, uint32_t lds_addr) __attribute__((always_inline)) {
        uint32_t tmp;
        asm volatile("s_mov_b32 m0, %1\n\tv_add_u32 %0, %2, %3\n\tglobal_load_lds_dwordx4 %0, %4"
                     : "=&v"(tmp)
                     : "s"(lds_addr), "v"(voff), "v"(vadd), "s"(base)
                     : "memory");
    };
    // load i of both panels of the group at the cursor (rows of the expanded weights hold whole groups: nothing to clamp)
    auto load_pair = [&](const int i, const uint32_t buf) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + buf + (uint32_t)(i * 64 * kRowBytes) + (uint32_t)wave * (8u * kRowBytes);
        if (i < WB) load16_to_lds(g.A.base, a_off[i], p_jb, dst);
        load16_to_lds(g.w_bytes, w_off[i], opaque(p_G * (uint32_t)kGroupK), dst + (uint32_t)kPanelBytes);
    };
    // Workgroup barrier: the next group has landed (its loads were issued a whole group ago) and this wave's LDS reads have
    // returned.
    auto panel_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // after the prologue: the first group has landed, the second may still be on its way
    auto first_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kLoadsPerGroup) : "memory");
    };

    // ------------------------------------------------------------------------------------------------ prologue
    p_locate();
    p_piece();
#pragma unroll
    for (int i = 0; i < 4; ++i) load_pair(i, 0u);
    p_advance();
#pragma unroll
    for (int i = 0; i < 4; ++i) load_pair(i, (uint32_t)kGroupBytes);
    first_barrier();

    uint32_t rd = 0u;  // byte offset of the group buffer being consumed

    // ------------------------------------------------------------------------------------------------ consumer
    // n_tiles tiles first_vb, first_vb + gridDim.x, ..., each wave multiplying WI blocks of 32 weight rows: two (the whole
    // tile) or one (half a tile), starting at weight row first_col of the panel.
    auto run_tiles = [&](auto wi_tag, const uint32_t first_vb, const uint32_t n_tiles, const uint32_t first_col) __attribute__((always_inline)) {
        constexpr int WI = decltype(wi_tag)::value;
        struct Frags {
            v4i a[WB], w[WI];
        };
        // Step s (0 .. 3) of a group: lane (r, kg) of a block holds the 16 elements k = 32 s + 16 kg .. + 15 of its row
        auto fetch = [&](const int s, const uint32_t buf, Frags &f) __attribute__((always_inline)) {
            const uint32_t ln = opaque(tid) & 63u;
            const uint32_t r = ln & 31u, kg = ln >> 5;
            const uint32_t piece = ((kg ^ ((r >> 1) & 7u)) << 4) ^ (uint32_t)(32 * s);
            const uint8_t *pa = lds + (buf + (uint32_t)(wm * 32 * WB * kRowBytes) + r * (uint32_t)kRowBytes + piece);
            const uint8_t *pw = lds + (buf + (uint32_t)kPanelBytes + (first_col + (uint32_t)(wn * 32 * WI) + r) * (uint32_t)kRowBytes + piece);
#pragma unroll
            for (int b = 0; b < WB; ++b) f.a[b] = *reinterpret_cast<const v4i *>(pa + b * 32 * kRowBytes);
#pragma unroll
            for (int b = 0; b < WI; ++b) f.w[b] = *reinterpret_cast<const v4i *>(pw + b * 32 * kRowBytes);
        };
        v16i acc[WI][WB];  // [n block][m block]
        int32_t ra[WB], rw[WI];
        auto multiply = [&](Frags &f) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < WB; ++j)
#pragma unroll
                for (int i = 0; i < WI; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.w[i], f.a[j], acc[i][j], 0, 0, 0);
        };
        Frags f0, f1;
        fetch(0, rd, f0);
        uint32_t vb = first_vb;
        for (uint32_t done = 0; done < n_tiles; ++done, vb += gridDim.x) {
            uint32_t tile_m, tile_n;
            tile_of_block(vb, total_tiles, tiles_m, tiles_n, tile_m, tile_n);
            const int64_t m_wave = (int64_t)tile_m * (64 * WB) + wm * 32 * WB, n_wave = (int64_t)tile_n * BN + (int64_t)first_col + wn * 32 * WI;
#pragma unroll
            for (int j = 0; j < WB; ++j) ra[j] = 0;
#pragma unroll
            for (int i = 0; i < WI; ++i) {
                rw[i] = 0;
#pragma unroll
                for (int j = 0; j < WB; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
            }
            for (uint32_t G = 0; G < ngroups; ++G) {
                const uint32_t other = rd ^ (uint32_t)kGroupBytes;
                p_advance();
                fetch(1, rd, f1);
                multiply(f0);
                __builtin_amdgcn_sched_barrier(0);
                fetch(2, rd, f0);
                multiply(f1);
                __builtin_amdgcn_sched_barrier(0);
                fetch(3, rd, f1);
                multiply(f0);
                __builtin_amdgcn_sched_barrier(0);
                panel_barrier();  // every wave holds the last step's operands: the buffer is free
#pragma unroll
                for (int i = 0; i < 4; ++i) load_pair(i, rd);
                fetch(0, other, f0);
                multiply(f1);
                __builtin_amdgcn_sched_barrier(0);
                rd = other;
            }
            // The sums are pinned here: otherwise the compiler moves matrix-core instructions down into the epilogue's blocks
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int j = 0; j < WB; ++j) asm volatile("" : "+v"(acc[i][j]));
            panel::wave_finish<false, WI, kLoadsPerGroup, panel::kNoTerms>(g, mc, acc, ra, rw, nullptr, nullptr, nullptr, stage_w, m_wave, n_wave);
        }
    };
    run_tiles(std::integral_constant<int, 2>{}, vb0, n_mine, 0u);
    if constexpr (kTail) {
        if (has_half) run_tiles(std::integral_constant<int, 1>{}, tail_vb, 1u, half_col);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads beyond the last tile)
}

typedef void (*KernelFn)(const GemmArgs, const MfmaConst, uint32_t, uint32_t, uint32_t);
// blocks: rows of a tile / 64 (four with tail)
KernelFn kernel_values(bool tail, int blocks);

}  // namespace bytes_panel
}  // namespace qnn
