// Wide variant of the panel-fed kernel (qnn_gemm_panel_kernel.h) for single-plane products with int32 sums that make whole rounds of
// large tiles: ONE workgroup on a compute unit, four waves of 128 x 128 on a 256 x 256 tile, one wave per SIMD.
//
// A wave of 128 x 128 makes three vector instructions per matrix-core instruction where one of 64 x 128 makes 4.6, so its main loop
// runs at 8.3 PTOP/s against 7.2 (at the card's lower clock under two busy waves a SIMD); nothing covers its barriers and its stores, 9.5
// us a round of 256 tiles.  8192^3, four rounds: 169 against 177 us; 8192 x 8192 x 16384 302 against 331, x 4096 103 and 103,
// x 1024 60 against 51; 7000 x 7000 x 7168, three rounds and a thin one, 148 against 129.
//   * The workgroup brings in whole 128-byte lines of the operand rows it shares, a group of four steps (128 bytes of every row: 64
//     KiB) at a time, with loads that write straight to LDS, each wave 16 of them per group, issued right after the barrier that frees a
//     group buffer, i.e. at least three steps (about 6000 cycles) before the data is needed; two group buffers take turns.
//   * A 16-byte piece c of row r sits at piece c xor (r / 2 mod 8) of its LDS row.
//   * Words become E2M1 operands as in gemm_panel_kernel; the shifts of the fourth phase are spread over the others, so that every
//     phase carries the same number of vector instructions.
//   * The one wave a SIMD holds issues every instruction itself, so whatever depends on the tile only (row offsets of the loads) is
//     worked out when the producer's cursor enters a tile.
// Requirements: as gemm_panel_kernel, rows of whole 128-byte groups.
#pragma once
#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"

namespace qnn {
namespace panel_wide {

using mfma::MfmaConst;
using mfma::v16f;
using mfma::v4i;
using mfma::v8i;

constexpr int kThreads = 256;
constexpr int WB = 4, WTILE = 128, BM = 256, BN = 256;
constexpr int kRowBytes = 128;                 // bytes of a row per group: four steps of two 16-byte k-groups
constexpr int kPanelBytes = BM * kRowBytes;    // one operand's 256 rows
constexpr int kGroupBytes = 2 * kPanelBytes;
constexpr int kGroupWords = kRowBytes / 4;

__device__ __forceinline__ uint32_t word_of(const uint4 &v, int t) { return t == 0 ? v.x : (t == 1 ? v.y : (t == 2 ? v.z : v.w)); }

// Schedule of one phase: 16 matrix-core instructions, each followed by its share of kValu vector-ALU instructions;
// kDsRead LDS reads behind the first matrix-core instructions, kDsWrite LDS writes and then kVmem global loads behind
// the following ones (one each).
template <int kValu, int kDsRead, int kDsWrite, int kVmem, int... I>
__device__ __forceinline__ void phase_groups(std::integer_sequence<int, I...>) {
    constexpr int n = (int)sizeof...(I);
    ((__builtin_amdgcn_sched_group_barrier(0x008, 1, 0),
      __builtin_amdgcn_sched_group_barrier(0x002, kValu / n + (I < kValu % n ? 1 : 0), 0),
      (I < kDsRead ? __builtin_amdgcn_sched_group_barrier(0x100, 1, 0) : (void)0),
      (I < kDsWrite ? __builtin_amdgcn_sched_group_barrier(0x200, 1, 0) : (void)0),
      (I >= kDsWrite && I < kDsWrite + kVmem ? __builtin_amdgcn_sched_group_barrier(0x020, 1, 0) : (void)0)),
     ...);
}

__global__ __launch_bounds__(kThreads, 1) void gemm_panel_wide_kernel(const GemmArgs g, const MfmaConst mc, uint32_t tiles_m, uint32_t tiles_n, uint32_t ngroups) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kGroupBytes];
    __shared__ __attribute__((aligned(16))) uint32_t rw_table[kThreads / 64][WTILE];
    // per wave one 32 x 32 staging block, through which a block is turned from the accumulator layout (a lane = one row) into whole
    // 128-byte lines per row
    __shared__ __attribute__((aligned(16))) int32_t stage[kThreads / 64][32 * 32];

    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    constexpr int kLoadsPerGroup = 16;  // loads to LDS that a wave issues per group
    const uint32_t total_tiles = tiles_m * tiles_n;

    // ------------------------------------------------------------------------------------------------ producer
    // A load instruction of a wave covers 8 consecutive rows x 128 bytes and fills 1 KiB of LDS: lane i lands at
    // 16 i behind the address in M0, i.e. in slot i mod 8 of row i / 8, so it fetches piece (i mod 8) xor (row / 2 mod 8).
    // Per quarter (64 rows) of a panel wave w loads rows 8 w .. 8 w + 7 and 32 + 8 w .. 32 + 8 w + 7.  Rows are
    // addressed by 32-bit byte offsets from the operand's base.
    // The lane-dependent parts are re-derived behind an opaque copy wherever they are used: address arithmetic that the
    // compiler computes once before the loops ends up spilled, and every reload in the main loop stalls the wave.
    auto opaque = [](uint32_t x) __attribute__((always_inline)) {
        asm volatile("" : "+v"(x));
        return x;
    };
    const uint32_t tid = (uint32_t)t;
    const uint32_t lds_base = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds);
    // The producer's cursor: tile p_vb, group p_G of its rows.  Everything that depends on the tile only (the byte
    // offsets of the rows this lane loads, with its piece of the line) is worked out when the cursor enters a tile,
    // under a branch of its own; per group only the scalar base pointers move on.  The one wave a SIMD holds issues
    // every instruction of the loop itself, so each instruction kept out of the groups is time won.
    // This workgroup's tiles: vb0, vb0 + gridDim.x, ... (n_mine of them).
    const uint32_t vb0 = blockIdx.x;
    const uint32_t n_mine = (total_tiles - vb0 + gridDim.x - 1u) / gridDim.x;
    uint32_t p_vb = vb0, p_G = 0, p_item = 0;
    // One register per panel holds the offset of the lane's row in the first 32-row block, a second one the offset in the operand's last
    // row, and a load adds its block's distance and clamps.
    uint32_t a_off = 0, w_off = 0, a_max = 0, w_max = 0;
    const uint32_t lda_bytes = (uint32_t)g.A.ld * 4u, ldw_bytes = (uint32_t)g.ldw * 4u;
    const uint32_t last_m = (uint32_t)(g.M - 1), last_n = (uint32_t)(g.N - 1);
    auto p_locate = [&]() __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(p_vb, total_tiles, tiles_m, tiles_n, tm, tn);
        const uint32_t tt = opaque(tid);
        const uint32_t pr = tt >> 3;                                  // row within a load's 32-row block
        const uint32_t piece16 = ((tt & 7u) ^ ((tt >> 4) & 7u)) << 4;  // (slot xor (row / 2 mod 8)) * 16 bytes
        // (the host checks that offsets up to one tile beyond the last row still fit 32 bits)
        a_off = (tm * (uint32_t)BM + pr) * lda_bytes + piece16;
        w_off = (tn * (uint32_t)BN + pr) * ldw_bytes + piece16;
        a_max = last_m * lda_bytes + piece16;
        w_max = last_n * ldw_bytes + piece16;
    };
    auto p_advance = [&]() __attribute__((always_inline)) {
        ++p_G;
        if (p_G == ngroups) {
            asm volatile("" ::: "memory");  // keeps the branch a branch
            p_G = 0;
            ++p_item;
            if (p_item < n_mine) p_vb = vb0 + p_item * gridDim.x;
            // (after the last tile the loads are repeated and never used)
            p_locate();
        }
    };
    // 16 bytes per lane from base + min(voff + sadd, vmax) to LDS address lds_addr + 16 * lane.  The address travels in M0; between the
    // write of M0 and the load there has to be an instruction, here the one that makes the offset.
    auto load_clamped_to_lds = [](const void *base, uint32_t voff, uint32_t sadd, uint32_t vmax, uint32_t lds_addr) __attribute__((always_inline)) {
        uint32_t tmp;
        asm volatile("s_mov_b32 m0, %1\n\tv_add_u32 %0, %3, %2\n\tv_min_u32 %0, %0, %4\n\tglobal_load_lds_dwordx4 %0, %5"
                     : "=&v"(tmp)
                     : "s"(lds_addr), "v"(voff), "s"(sadd), "v"(vmax), "s"(base)
                     : "memory");
    };
    // quarter q (rows 64 q .. 64 q + 63 of both panels) of the group at the cursor into the group buffer at byte offset buf
    auto load_quarter = [&](const int q, const uint32_t buf) __attribute__((always_inline)) {
        const uint8_t *a_base = reinterpret_cast<const uint8_t *>(g.A.base) + p_G * (uint32_t)kRowBytes;
        const uint8_t *w_base = reinterpret_cast<const uint8_t *>(g.W) + p_G * (uint32_t)kRowBytes;
        const uint32_t dst = lds_base + buf + (uint32_t)(q * (64 * kRowBytes)) + (uint32_t)wave * (8u * kRowBytes);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = 2 * q + h;
            load_clamped_to_lds(a_base, a_off, (uint32_t)(32 * i) * lda_bytes, a_max, dst + (uint32_t)(h * 32 * kRowBytes));
            load_clamped_to_lds(w_base, w_off, (uint32_t)(32 * i) * ldw_bytes, w_max, dst + (uint32_t)(kPanelBytes + h * 32 * kRowBytes));
        }
    };

    // workgroup barrier of the group buffers: this wave's loads to LDS have landed and its LDS reads have returned
    auto panel_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // after the prologue: the first group has landed (the second may still be on its way: every workgroup asks for its first groups at
    // the same moment, and waiting for all of them costs microseconds per launch)
    auto first_barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kLoadsPerGroup) : "memory"); };

    // ------------------------------------------------------------------------------------------------ prologue
    // the first groups into the buffers; the cursor stays at the last of them
    p_locate();
#pragma unroll 1
    for (int b = 0; b < 2; ++b) {
        if (b > 0) p_advance();
#pragma unroll
        for (int q = 0; q < 4; ++q) load_quarter(q, (uint32_t)(b * kGroupBytes));
    }
    first_barrier();

    uint32_t rd = 0u;  // byte offset of the group buffer being consumed
    auto no_produce = [](auto) __attribute__((always_inline)) {};
    // Fourth step of a group (after the barrier, the buffer just consumed is free): phase t starts the loads of
    // quarter t of the group two groups ahead into it.
    auto produce = [&](auto t_tag) __attribute__((always_inline)) {
        constexpr int tt = decltype(t_tag)::value;
        load_quarter(tt, rd);
    };

    // ------------------------------------------------------------------------------------------------ consumer
    constexpr int kMfma = WB * WB;  // matrix-core instructions of a phase
    // lane (r, kg) of block b reads piece 2 q + kg of row 32 b + r at step q of a group
    struct Step {
        uint4 A[WB], W[WB];
    };
    auto fetch = [&](const int q, const uint32_t buf, Step &d) __attribute__((always_inline)) {
        const uint32_t ln = opaque(tid) & 63u;
        const uint32_t r = ln & 31u, kg = ln >> 5;
        const uint32_t piece = ((kg ^ ((r >> 1) & 7u)) << 4) ^ (uint32_t)(q << 5);
        const uint8_t *pa = lds + (buf + (uint32_t)(wm * WTILE * kRowBytes) + r * (uint32_t)kRowBytes + piece);
        const uint8_t *pw = lds + (buf + (uint32_t)kPanelBytes + (uint32_t)(wn * WTILE * kRowBytes) +
                                   r * (uint32_t)kRowBytes + piece);
#pragma unroll
        for (int b = 0; b < WB; ++b) d.A[b] = *reinterpret_cast<const uint4 *>(pa + b * (32 * kRowBytes));
#pragma unroll
        for (int b = 0; b < WB; ++b) d.W[b] = *reinterpret_cast<const uint4 *>(pw + b * (32 * kRowBytes));
    };

    v16f acc[WB][WB];  // [n block][m block]
    int32_t ra[WB], rw[WB];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < WB; ++j) ra[j] = 0;
#pragma unroll
        for (int i = 0; i < WB; ++i) {
            rw[i] = 0;
#pragma unroll
            for (int j = 0; j < WB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        }
    };
    // An E2M1 operand of the instruction is four registers; the builtin's operand type has eight, of which the upper
    // four are left undefined (the instruction does not read them in this format), so that they occupy nothing.
    struct Frags {
        v4i a[WB], w[WB];
    };
    auto widen = [](const v4i &x) __attribute__((always_inline)) { return __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1); };
    // Phase t of a step multiplies bit t of every nibble of the lane's four words (32 of its 128 elements of k; both
    // operands use the same order).  An E2M1 nibble with only bit 0 set is 0.5, with bit 1 set 1.0, with bit 2 set 2.0,
    // so for t = 0, 1, 2 one AND per word makes the operand and the block scale of the instruction (2, 1, 1/2 on
    // both sides: exact powers of two) turns every product of two set bits into 1; bit 3 is the sign and is moved to
    // bit 1 first.  20 vector-ALU instructions per 128 elements instead of 28 with shift-and-mask throughout.
    auto expand = [&](const Step &c, const int tt, Frags &f) __attribute__((always_inline)) {
        const uint32_t mask = tt == 0 ? 0x11111111u : (tt == 2 ? 0x44444444u : 0x22222222u);
#pragma unroll
        for (int b = 0; b < WB; ++b) {
#pragma unroll
            for (int j = 0; j < 4; ++j) f.a[b][j] = (int)(word_of(c.A[b], j) & mask);
        }
#pragma unroll
        for (int b = 0; b < WB; ++b) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f.w[b][j] = (int)(word_of(c.W[b], j) & mask);
            }
        }
    };
    // Bit 3 of a nibble takes two instructions per word (shift, mask).  The shifts are spread over the three phases
    // before the one that needs them (word number idx of the step in phase idx mod 3), so that every phase carries about
    // the same number of vector-ALU instructions: a phase that carries more than its matrix-core instructions cover
    // stalls the one wave of the SIMD.
    struct Shifted {
        uint32_t a[WB][4], w[WB][4];
    };
    auto shift_part = [&](const Step &c, const int part, Shifted &sh) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((b * 4 + j) % 3 == part) sh.a[b][j] = word_of(c.A[b], j) >> 2;
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((WB * 4 + b * 4 + j) % 3 == part) sh.w[b][j] = word_of(c.W[b], j) >> 2;
    };
    auto expand_shifted = [&](const Step &c, const Shifted &sh, Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < WB; ++b) {
#pragma unroll
            for (int j = 0; j < 4; ++j) f.a[b][j] = (int)(sh.a[b][j] & 0x22222222u);
        }
#pragma unroll
        for (int b = 0; b < WB; ++b) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f.w[b][j] = (int)(sh.w[b][j] & 0x22222222u);
            }
        }
    };
    // row sums of the raw bits: one word of every row per phase.  Each sum is made opaque after its addition: left
    // alone, the compiler keeps the counts of a whole loop trip in registers of their own and adds them up at the end
    // (three-operand adds), which costs over a hundred registers and spills the sums themselves.
    auto count = [&](const Step &c, const int tt) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            ra[b] += (int32_t)__builtin_popcount(word_of(c.A[b], tt));
            asm("" : "+v"(ra[b]));
        }
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            rw[b] += (int32_t)__builtin_popcount(word_of(c.W[b], tt));
            asm("" : "+v"(rw[b]));
        }
    };
    // block scales of the four phases as E8M0 bytes (2^(e - 127)): 2, 1, 1/2, 1
    const int scales = 0x7F7E7F80;
    auto multiply = [&](const Frags &f, auto t_tag) __attribute__((always_inline)) {
        constexpr int tt = decltype(t_tag)::value;
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int j = 0; j < WB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(widen(f.w[i]), widen(f.a[j]), acc[i][j], 4, 4, tt, scales, tt, scales);
    };
    // One step = four phases; each phase multiplies the operands made during the previous one and meanwhile counts
    // one word per row and makes the next phase's operands.  `issue_fetch` (the LDS reads of the following step) runs
    // inside the first phase; `produce(t)` is called in every phase (the fourth step of a group uses it to start the
    // loads of a quarter of the group after the next).
    auto compute = [&](const Step &c, const Step &n, Frags &f, auto issue_fetch, auto produce,
                       auto last_tag) __attribute__((always_inline)) {
        constexpr bool kLastStep = decltype(last_tag)::value;
        Shifted sh;
        auto phase = [&](auto t_tag) __attribute__((always_inline)) {
            constexpr int tt = decltype(t_tag)::value;
            if (tt == 0) issue_fetch();
            produce(t_tag);
            Frags gnext;
            // counts: word t in phases 0, 1 and 3; word 2 in phase 3 as well (phase 2 carries shifts instead)
            if (tt != 2) count(c, tt);
            if (tt == 3) count(c, 2);
            if (tt < 3) shift_part(c, tt, sh);
            if (tt + 1 < 3)
                expand(c, tt + 1, gnext);
            else if (tt == 2)
                expand_shifted(c, sh, gnext);
            else if (!kLastStep)
                expand(n, 0, gnext);
            multiply(f, t_tag);
            // vector-ALU instructions of this phase: 4 masks per row, its share of the shifts and of the counts
            constexpr int kRows = WB + WB;
            constexpr int kShifts = tt < 3 ? (4 * kRows + 2 - tt) / 3 : 0;
            constexpr int kOps = kRows * 4 + kShifts + (tt == 2 ? 0 : (tt == 3 ? 2 * kRows : kRows));
            if (tt == 0)
                phase_groups<kOps + 8, WB + WB, 0, 0>(std::make_integer_sequence<int, kMfma>{});
            else
                phase_groups<kOps, 0, 0, 0>(std::make_integer_sequence<int, kMfma>{});
            __builtin_amdgcn_sched_barrier(0);
            if (!(kLastStep && tt == 3)) f = gnext;
        };
        phase(std::integral_constant<int, 0>{});
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
    };

    auto finish = [&](const int64_t m_wave, const int64_t n_wave) __attribute__((always_inline)) {
        panel::wave_finish<false, WB, kLoadsPerGroup, panel::kBothTerms>(g, mc, acc, ra, rw, rw_table[wave], nullptr, nullptr, stage[wave], m_wave, n_wave);
    };

    Step buf0, buf1;
    Frags frags;
    fetch(0, rd, buf0);
    expand(buf0, 0, frags);

    uint32_t vb = vb0;
    for (uint32_t done = 0; done < n_mine; ++done, vb += gridDim.x) {
        uint32_t tile_m, tile_n;
        tile_of_block(vb, total_tiles, tiles_m, tiles_n, tile_m, tile_n);
        const int64_t m_wave = (int64_t)tile_m * BM + wm * WTILE;
        const int64_t n_wave = (int64_t)tile_n * BN + wn * WTILE;
        clear();
        // one group of four steps; last_tag: its last step ends the tile
        auto group = [&](auto last_tag) __attribute__((always_inline)) {
            const uint32_t other = rd ^ (uint32_t)kGroupBytes;
            // the cursor moves on to the group that this group's fourth step will load (scalar control flow: kept at
            // the head of the group, so that the phases of a step stay one straight-line block)
            p_advance();
            compute(buf0, buf1, frags, [&]() __attribute__((always_inline)) { fetch(1, rd, buf1); }, no_produce, std::false_type{});
            compute(buf1, buf0, frags, [&]() __attribute__((always_inline)) { fetch(2, rd, buf0); }, no_produce, std::false_type{});
            compute(buf0, buf1, frags, [&]() __attribute__((always_inline)) { fetch(3, rd, buf1); }, no_produce, std::false_type{});
            panel_barrier();
            // last step of the tile: the operands of the next tile's first phase are made after the epilogue, so that
            // they do not occupy registers during it
            compute(buf1, buf0, frags, [&]() __attribute__((always_inline)) { fetch(0, other, buf0); }, produce, last_tag);
            rd = other;
        };
        for (uint32_t G = 0; G + 1 < ngroups; ++G) group(std::false_type{});
        group(std::true_type{});
        finish(m_wave, n_wave);
        expand(buf0, 0, frags);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads beyond the last tile)
}

}  // namespace panel_wide
}  // namespace qnn
