// Matrix-core kernel for a left operand of small integers and a right operand of +-1 weights given as bits (the two products of the
// backward step, Alg. 1 with Sec. 5's quantized gradients).
//
// A log-quantized gradient is a power of two, so it is an FP6 (E3M2) number as it stands, and v_mfma_scale_f32_32x32x64_f8f6f4
// multiplies FP6 by FP4 in 32 cycles where the int8 instruction takes 64 for the same products: 7.4 against 4.2 PTOP/s with such
// operands and nothing else to do.  Where a value is not an E3M2 number (more than three leading bits), the operand's image
// holds int8 instead and the kernel takes its int8 branch; which of the two it is, the kernel that writes the images has decided on
// the data (qnn_gemm_mixed.hip).
//   Sums: an E3M2 code of n / 16 with the block scale 2^4 is the integer n, all products are integers up to 2^7 and the host keeps
// every sum within 2^24, where the instruction's float accumulation is exact.  In the int8 branch the weights are n = 0 / 1 for +1 / -1:
// sum g w = sum g - 2 sum g n.
//
// Operand images, in groups of k, so that a tile's part of a group is a few contiguous ranges, copied to LDS as they lie with loads of
// 1024 bytes that need no address arithmetic per lane; the places of the pieces put the lanes that an LDS read serves together on
// different banks:
//   FP6, groups of 256: low [group][row][8 pieces of 16 bytes], piece c holds the first four words of the 32 elements 32 c .. + 31 (six
//     words), at place c xor (row / 2 mod 8); high [group][step][row][2 x 8 bytes], the last two words of pieces c = 4 h + step, at
//     place h xor (row / 16 mod 2).
//   int8, groups of 128: [group][row][8 pieces of 16 elements], piece c at place c xor (row / 2 mod 8), elements of every eight in the
//     order 0 2 4 6 1 3 5 7.
//   bits, groups of 128: [group][row][4 words]; bit t of nibble j of word i is the INVERTED bit of element 32 t + 8 i + j, so that
//     step t finds its operand in bit t of every nibble: shifted to the sign position and combined with 0x2 it is the E2M1 value +-1
//     (two instructions per register); every other nibble's bit at the bottom of a byte is an int8 value 0 / 1.
//   A tile at the lower edge reads rows that are not the group's (its results there are not stored); they lie in the group behind it, or in
//   room behind the last one (see values_bytes).  Elements of k beyond the last are zero values.
// Workgroup: four waves on a tile of 32 MB WM x 32 NB (4 / WM), two group buffers behind one barrier per group, and TWO workgroups on a
// compute unit, so that one multiplies while the other waits at its barrier or stores its tile: 128 x 256 tiles, 10000 x 4096 x 4096, 93 us
// against 107 of one workgroup of eight waves with the same waves on 256 x 256 (4096 x 4096 x 10000 87 against 103; int8 136 against 155,
// and against 135 - 160 of both operands as int8 in LDS).  Weights as bits keep LDS reads at half of what the matrix cores leave
// time for and cost 3.5 vector instructions per matrix-core instruction.  What bounds it: power (on zeros 66 and 63 us, at a higher clock).
#pragma once
#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_panel_epilogue.h"

namespace qnn {
namespace mixed {

using mfma::MfmaConst;
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kFlags = 512;  // words that say whether some value is not an E3M2 number

struct MixedArgs {
    const uint8_t *a, *w;             // images
    const uint32_t *inexact;          // [kFlags]: int8 image if any is set
    uint32_t rows_a, rows_w;          // rows of an image's group
    uint32_t groups, halves;          // of 256 elements, of 128 (int8)
    Tiles tiles;
    int32_t alpha;                    // C = alpha S
    int alpha_shift;                  // alpha = 2^alpha_shift, or -1
};

template <bool kBytes, int kWaves, int MB, int NB, int WM>
__device__ __forceinline__ void product(const GemmArgs &g, const MixedArgs &x, uint8_t *const lds) {
    constexpr int WN = kWaves / WM, BM = 32 * MB * WM, BN = 32 * NB * WN;
    // a group in LDS: FP6 low, FP6 high or int8; then the bits
    constexpr uint32_t kLow = BM * 128, kHighStep = kBytes ? 0 : BM * 16, kHigh = 4 * kHighStep, kBits = kBytes ? BN * 16 : 2 * BN * 16;
    constexpr uint32_t kGroup = kLow + kHigh + kBits;
    const uint32_t lane = threadIdx.x & 63u, r = lane & 31u, kg = lane >> 5;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave / WN, wn = wave % WN;
    const uint32_t total = x.tiles.total, groups = kBytes ? x.halves : x.groups;
    // (where the loads ahead of the loop may enter a second tile, the code in front of the loop grows and the int8 loop, unchanged, runs
    // 5 % slower: 8111 x 1008 x 638, second product, 40.8 against 42.9 us)
    if constexpr (kBytes) __builtin_assume(groups >= 2u);
    const uint32_t lds_base = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds);
    int32_t *const stage_w = reinterpret_cast<int32_t *>(lds + 2 * kGroup + wave * 4096);
    auto opaque = [](uint32_t v) __attribute__((always_inline)) {
        asm volatile("" : "+v"(v));
        return v;
    };

    // ------------------------------------------------------------------------------------------------ producer
    // The producer's cursor (a tile, group p_G) runs two groups ahead of the multiplication; the pointers are this wave's.
    const uint32_t vb0 = blockIdx.x;
    const uint32_t n_mine = (total - vb0 + gridDim.x - 1u) / gridDim.x;
    uint32_t p_G = 0, p_item = 0;
    const uint8_t *p_low, *p_high, *p_bits;
    const uint8_t *const high_image = x.a + (uint64_t)x.groups * x.rows_a * 128u;
    // pieces of 1024 bytes are dealt out to the waves: of low by eights, of high and the bits as below
    constexpr uint32_t kHighPieces = kHigh / 1024u, kHighPerStep = kHighStep ? kHighStep / 1024u : 1u, kBitPieces = kBits / 1024u, kBitPerGroup = BN * 16 / 1024u;
    auto p_locate = [&](const uint32_t vb) __attribute__((always_inline)) {
        uint32_t tm, tn;
        tile_of_block(vb, x.tiles, tm, tn);
        p_low = x.a + (uint64_t)tm * (BM * 128u) + wave * 1024u;
        p_high = high_image + (uint64_t)tm * (BM * 16u);
        p_bits = x.w + (uint64_t)tn * (BN * 16u);
    };
    auto p_advance = [&]() __attribute__((always_inline)) {
        p_low += (uint64_t)x.rows_a * 128u, p_high += (uint64_t)x.rows_a * 64u;
        p_bits += (uint64_t)x.rows_w * (kBytes ? 16u : 32u);
        if (++p_G == groups) {
            asm volatile("" ::: "memory");  // keeps the branch a branch
            p_G = 0;
            ++p_item;
            // (after the last tile the loads start over and are never used)
            p_locate(p_item < n_mine ? vb0 + p_item * gridDim.x : vb0);
        }
    };
    // 1024 bytes from base to LDS address dst, 16 per lane
    const uint32_t lane16 = lane * 16u;
    auto load1k = [&](const uint8_t *base, const uint32_t dst) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(lane16), "s"(base) : "memory");
    };
    // part 0 .. kParts - 1 of the loads of the group at the cursor into the buffer at `buf`
    constexpr int kLowLoads = kLow / 1024 / kWaves, kHighLoads = (kHighPieces + kWaves - 1) / kWaves, kBitLoads = (kBitPieces + kWaves - 1) / kWaves;
    constexpr int kParts = kLowLoads + kHighLoads + kBitLoads;
    static_assert(kLow / 1024 % kWaves == 0, "whole rounds of loads");
    auto load_part = [&](const int part, const uint32_t buf) __attribute__((always_inline)) {
        const uint32_t dst = lds_base + buf;
        if (part < kLowLoads) {
            load1k(p_low + part * (1024 * kWaves), dst + (part * kWaves + wave) * 1024u);
        } else if (part < kLowLoads + kHighLoads) {
            const uint32_t piece = kWaves * (part - kLowLoads) + wave, step = piece / kHighPerStep, at = piece % kHighPerStep;
            if (kHighPieces % kWaves == 0u || piece < kHighPieces) load1k(p_high + (uint64_t)step * x.rows_a * 16u + at * 1024u, dst + kLow + piece * 1024u);
        } else {
            const uint32_t piece = kWaves * (part - kLowLoads - kHighLoads) + wave, half = piece / kBitPerGroup, at = piece % kBitPerGroup;
            if (kBitPieces % kWaves == 0u || piece < kBitPieces) load1k(p_bits + (uint64_t)half * x.rows_w * 16u + at * 1024u, dst + kLow + kHigh + piece * 1024u);
        }
    };
    // the next group has landed (its loads were issued a whole group ago) and this wave's LDS reads have returned
    auto barrier = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    p_locate(vb0);
#pragma unroll
    for (int i = 0; i < kParts; ++i) load_part(i, 0u);
    barrier();
    p_advance();
#pragma unroll
    for (int i = 0; i < kParts; ++i) load_part(i, kGroup);
    uint32_t rd = 0u;  // the group buffer being multiplied

    // ------------------------------------------------------------------------------------------------ consumer
    typedef std::conditional_t<kBytes, v16i, v16f> Acc;
    struct Values {
        v4i lo[MB];
        v2i hi[MB];
    };
    struct Words {
        std::conditional_t<kBytes, v2i, v4i> w[NB];  // int8: words 2 kg and 2 kg + 1 of the four
    };
    // step t: 32 elements of each half of a group of 256, or of a group of 128 (lane (r, kg): elements 16 kg .. + 15 of them)
    auto fetch_values = [&](const uint32_t t, const uint32_t buf, Values &f) __attribute__((always_inline)) {
        const uint32_t row = wm * (32u * MB) + r;  // (blocks of 32 rows do not change the places)
        const uint32_t piece = kBytes ? 2u * t + kg : 4u * kg + t;
        const uint8_t *const lo = lds + (buf + row * 128u + ((piece ^ ((r >> 1) & 7u)) << 4));
#pragma unroll
        for (int b = 0; b < MB; ++b) f.lo[b] = *reinterpret_cast<const v4i *>(lo + b * 32 * 128);
        if constexpr (!kBytes) {
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                // (apart for the compiler: one read for two blocks would leave their words in the wrong registers)
                const uint32_t hi = opaque(buf + kLow + t * kHighStep + (row + 32u * b) * 16u + ((kg ^ ((r >> 4) & 1u)) << 3));
                f.hi[b] = *reinterpret_cast<const v2i *>(lds + hi);
            }
        }
    };
    auto fetch_words = [&](const uint32_t buf, Words &f) __attribute__((always_inline)) {
        const uint8_t *const p = lds + (buf + kLow + kHigh + kg * (kBytes ? 8u : BN * 16u) + (wn * (32u * NB) + r) * 16u);
#pragma unroll
        for (int b = 0; b < NB; ++b) f.w[b] = *reinterpret_cast<const decltype(f.w[b] + 0) *>(p + b * 32 * 16);
    };
    Acc acc[NB][MB];  // [n block][m block]
    int32_t ra[MB];
    const uint32_t one = opaque(0x22222222u);
    // the products of weight block i with the values of step t
    auto multiply = [&](auto step_tag, const int i, const Values &f, const Words &z) __attribute__((always_inline)) {
        constexpr int t = decltype(step_tag)::value;
        v4i w;
        if constexpr (kBytes) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // elements 16 kg + 8 (e / 2) + (e mod 2) + 0, 2, 4, 6
                w[e] = (int)(((uint32_t)z.w[i][e >> 1] >> (4 * (e & 1) + t)) & 0x01010101u);
            }
#pragma unroll
            for (int j = 0; j < MB; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, f.lo[j], acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (int)((((uint32_t)z.w[i][e] << (3 - t)) & 0x88888888u) | one);
            const v8i w8 = __builtin_shufflevector(w, w, 0, 1, 2, 3, -1, -1, -1, -1);
#pragma unroll
            for (int j = 0; j < MB; ++j) {
                const v4i h4 = __builtin_shufflevector(f.hi[j], f.hi[j], 0, 1, -1, -1);
                const v8i a = __builtin_shufflevector(f.lo[j], h4, 0, 1, 2, 3, 4, 5, -1, -1);
                // formats: 4 = E2M1, 3 = E3M2; scales 2^0 and 2^4
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w8, a, acc[i][j], 4, 3, 0, 0x7F7F7F7F, 0, (int)0x83838383u);
            }
        }
    };
    auto step = [&](auto step_tag, const Values &f, const Words &z) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NB; ++i) multiply(step_tag, i, f, z);
        if constexpr (kBytes) {  // the values' sums
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) ra[j] = __builtin_amdgcn_sdot4(f.lo[j][e], 0x01010101, ra[j], false);
        }
    };
    std::integral_constant<int, 0> s0;
    std::integral_constant<int, 1> s1;
    std::integral_constant<int, 2> s2;
    std::integral_constant<int, 3> s3;

    MfmaConst mc;
    mc.alpha = (uint32_t)(kBytes ? -2 * x.alpha : x.alpha), mc.alpha_shift = kBytes ? -1 : x.alpha_shift;
    mc.cRA = kBytes ? (uint32_t)x.alpha : 0u, mc.cRW = mc.c0 = 0u, mc.needRW = 0;
    Values f0, f1;
    Words z, zn;
    fetch_values(0, rd, f0);
    fetch_words(rd, z);
    uint32_t vb = vb0;
    for (uint32_t done = 0; done < n_mine; ++done, vb += gridDim.x) {
        uint32_t tile_m, tile_n;
        tile_of_block(vb, x.tiles, tile_m, tile_n);
        const int64_t m_wave = (int64_t)tile_m * BM + wm * (32 * MB), n_wave = (int64_t)tile_n * BN + wn * (32 * NB);
#pragma unroll
        for (int j = 0; j < MB; ++j) ra[j] = 0;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
        // (the scheduling barriers keep a step's reads ahead of the products of the step before)
        for (uint32_t G = 0; G < groups; ++G) {
            const uint32_t other = kGroup - rd;
            p_advance();
            fetch_values(1, rd, f1);
            __builtin_amdgcn_sched_barrier(0);
            step(s0, f0, z);
            __builtin_amdgcn_sched_barrier(0);
            fetch_values(2, rd, f0);
            __builtin_amdgcn_sched_barrier(0);
            step(s1, f1, z);
            __builtin_amdgcn_sched_barrier(0);
            fetch_values(3, rd, f1);
            __builtin_amdgcn_sched_barrier(0);
            step(s2, f0, z);
            __builtin_amdgcn_sched_barrier(0);
            barrier();  // every wave holds the last step's operands: the buffer is free
            fetch_values(0, other, f0);
            fetch_words(other, zn);
            __builtin_amdgcn_sched_barrier(0);
            // the last step's products, and between them the loads two groups ahead
            constexpr int kEach = (kParts + NB - 1) / NB;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                multiply(s3, i, f1, z);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < kEach; ++p)
                    if (kEach * i + p < kParts) load_part(kEach * i + p, rd);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (kBytes) {
#pragma unroll
                for (int j = 0; j < MB; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) ra[j] = __builtin_amdgcn_sdot4(f1.lo[j][e], 0x01010101, ra[j], false);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) z.w[i] = zn.w[i];
            rd = other;
        }
        // The sums are pinned here: otherwise the compiler moves matrix-core instructions down into the epilogue's blocks
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) asm volatile("" : "+v"(acc[i][j]));
        int32_t rw[NB] = {};
        panel::wave_finish<false, NB, 0, kBytes ? panel::kRowTerms : panel::kNoTerms>(g, mc, acc, ra, rw, nullptr, nullptr, nullptr, stage_w, m_wave, n_wave);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads beyond the last tile)
}

template <int kWaves, int MB, int NB, int WM>
__global__ __launch_bounds__(64 * kWaves, 2) void gemm_mixed_kernel(const GemmArgs g, const MixedArgs x) {
    constexpr int BM = 32 * MB * WM, BN = 32 * NB * (kWaves / WM);
    constexpr int kBuffers = 2 * (BM * 192 + BN * 32) + kWaves * 4096;  // two FP6 groups (the larger ones), a staging block per wave
    static_assert(kBuffers <= 160 * 1024, "LDS of a compute unit");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kBuffers];
    static_assert(kFlags == 512, "eight words a lane");
    const uint4 *const flags = reinterpret_cast<const uint4 *>(x.inexact) + 2 * (threadIdx.x & 63u);
    const uint4 f0 = flags[0], f1 = flags[1];
    if (__any((int)(f0.x | f0.y | f0.z | f0.w | f1.x | f1.y | f1.z | f1.w)))
        product<true, kWaves, MB, NB, WM>(g, x, lds);
    else
        product<false, kWaves, MB, NB, WM>(g, x, lds);
}

}  // namespace mixed
}  // namespace qnn
