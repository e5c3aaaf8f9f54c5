// Epilogues of the panel-fed matrix-core kernels: what a wave does with its finished accumulators.
//   int32 sums: C = alpha S + cRA RA[m] + cRW RW[n] + c0 (the rank-one correction that turns the product of raw codes
//   into the product of the values they stand for), every 32 x 32 block passed through a per-wave LDS block so that it
//   leaves as whole 128-byte lines;
//   threshold: bit = (C >= T[n]) xor flip[n] (Alg. 4: a^b = Sign(BatchNorm(a)) with BatchNorm folded to an integer
//   threshold), packed along n.
#pragma once
#include "qnn_gemm_mfma_kernel.h"

namespace qnn {
namespace panel {

using mfma::acc_to_sum;
using mfma::i32x4;
using mfma::MfmaConst;
using mfma::or_halves;
using mfma::sum_halves;

// Thresholds T[n] (int32) and flip flags flip[n] (uint8, may be absent) of the wave's columns n_wave .. + 32 WBN - 1
// (clamped to the last column) straight into the wave's LDS tables, one entry per lane and load, without passing
// through registers: a load into registers would make the compiler wait for every outstanding memory operation,
// among them the operand loads of the following groups, before the first use of the value.  If there are no flip flags
// the table keeps the zeros it was cleared to at the start of the kernel.
template <int WBN>
__device__ __forceinline__ void load_thresholds_to_lds(const GemmArgs &g, const int64_t n_wave, int32_t *thr_tab,
                                                       uint32_t *flip_tab) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t thr_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) int32_t *)thr_tab);
    const uint32_t flip_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t *)flip_tab);
#pragma unroll
    for (int h = 0; h < (WBN + 1) / 2; ++h) {
        int64_t n = n_wave + 64 * h + lane;
        if (n > g.N - 1) n = g.N - 1;
        const uint32_t off = (uint32_t)n;  // (N < 2^31)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(thr_lds + 256u * h), "v"(off * 4u), "s"(g.epi.T) : "memory");
        if (g.epi.flip)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ubyte %1, %2" : : "s"(flip_lds + 256u * h), "v"(off), "s"(g.epi.flip) : "memory");
    }
}

// A lane's words of 32 columns (n_wave + 32 i ..) of row m, the last of a row's columns cut off where they end.
template <int WBN>
__device__ __forceinline__ void store_words(const GemmArgs &g, const uint32_t (&word)[WBN], const int64_t m, const int64_t n_wave) {
    if (m >= g.M) return;
    uint32_t *const dst = g.epi.out_bits + m * g.epi.ldo + n_wave / 32;
    if (WBN == 4 && n_wave + 128 <= g.N && g.epi.ldo % 4 == 0 && reinterpret_cast<uintptr_t>(g.epi.out_bits) % 16 == 0) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(word[0], word[1], word[WBN - 2], word[WBN - 1]);
        return;
    }
#pragma unroll
    for (int i = 0; i < WBN; ++i) {
        const int64_t left = g.N - (n_wave + 32 * i);
        if (left > 0) dst[i] = left >= 32 ? word[i] : word[i] & ((1u << left) - 1u);
    }
}

// Accumulator register v of block [bi][bj] is C[m][n] with
//   m = m_wave + 32 bj + (lane mod 32),   n = n_wave + 32 bi + 8 (v / 4) + 4 (lane / 32) + v mod 4.
// kTile: kInside, the wave tile lies completely inside C and C allows 16-byte stores, so nothing needs a bounds check; kLower (int32
// sums), the same but for rows beyond the last; kAny, anything else.
// kTerms: which row sums C depends on.  kForm: how it is computed from the accumulators.
//   kUnits (float sums, coefficients +-1, so that everything stays far below 2^22): sums in single precision, where all these integers are
//     exact.  Thresholds: the sign of fma(-alpha, S, T - 1 - column term) - row term.  Int32: fma(alpha, S, column term + 3 2^22) has the
//     integer in its bits, and one integer addition takes the bits of 3 2^22 off and the row term on.  Three and two instructions per
//     element instead of five and three (thresholds, 10000 x 4096 x 4096 56.5 -> 54.2 us, 1999 x 3001 x 2500 12.0 -> 11.2).  Not in the widest
//     tile, whose registers are full (8192^3 180 -> 190).
//   kShift: alpha = 2^alpha_shift;  kTimes: any alpha.
// ra, rw: this lane's partial row sums of the raw codes (activation rows / weight rows of the wave tile); rw_tab,
// thr_tab, flip_tab (128 entries each) and stage_w (32 x 32 int32) are this wave's LDS areas.  thr_tab / flip_tab
// arrive holding the thresholds and flip flags (0 / non-zero) of columns n_wave .. n_wave + 32 WBN - 1, brought in by
// loads that write straight to LDS (see load_thresholds_to_lds) and that were followed by kLoadsAfter further loads
// of the same kind: waiting until at most that many loads are outstanding means the tables have landed, while the
// operand loads for the next tile stay in flight.
enum TileKind { kInside, kLower, kAny };
enum Terms { kNoTerms, kRowTerms, kBothTerms };
enum Form { kUnits, kShift, kTimes };
constexpr float kMagic = 12582912.0f;  // 3 2^22: adding it leaves an integer up to 2^22 in the low bits
constexpr uint32_t kMagicBits = 0x4B400000u;
template <bool kSign, int WBN, TileKind kTile, int kLoadsAfter, Terms kTerms, Form kForm, int WB, typename Acc>
__device__ __forceinline__ void wave_epilogue(const GemmArgs &g, const MfmaConst &mc, Acc (&acc)[WBN][WB], int32_t (&ra)[WB],
                                              int32_t (&rw)[WBN], uint32_t *rw_tab, int32_t *thr_tab, uint32_t *flip_tab,
                                              int32_t *stage_w, const int64_t m_wave, const int64_t n_wave) {
    constexpr int WTN = 32 * WBN;
    constexpr bool kFast = kTile != kAny;
    // The edge of C goes through LDS too, except in the widest tile, whose registers are full: there it made the whole kernel 0.5 %
    // slower (8192^3, which has no edge: 180.7 -> 181.6 us)
    constexpr bool kScatterEdge = WBN * WB == 16;
    static_assert(!kSign || kTerms == kBothTerms, "thresholds: both row sums");

    // lane coordinates re-derived behind an opaque copy: index arithmetic computed before the tile loop and kept
    // across it would be spilled, and a reload waits for every store issued before it
    int lane_opaque = (int)(threadIdx.x & 63);
    asm volatile("" : "+v"(lane_opaque));
    const int lane = lane_opaque, r = lane & 31, kg = lane >> 5;
    if constexpr (kTerms != kNoTerms) {
#pragma unroll
        for (int b = 0; b < WB; ++b) ra[b] = sum_halves(ra[b]);
    }
    if constexpr (kTerms == kBothTerms) {
#pragma unroll
        for (int b = 0; b < WBN; ++b) rw[b] = sum_halves(rw[b]);
    }
    // the column terms of C: lane l has those of columns l, 64 + l, ...
    auto column_term = [&](const int h) __attribute__((always_inline)) { return mc.cRW * (uint32_t)(kg ? rw[2 * h + 1] : rw[2 * h]); };
    const float alpha = (float)(int32_t)mc.alpha;
    if constexpr (kSign) {
        // thresholds, clamped and minus one, less the column terms, and flip flags at the bit position their n has in a lane's partial
        // output word (n mod 32 = 8 q + 4 kg + i  ->  bit 8 q + i): the per-wave LDS tables are rewritten in place.  Clamping at a bound
        // that |C| does not reach (2^22 - 2^20 with unit coefficients, 2^30 otherwise) changes no comparison.
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"(kLoadsAfter) : "memory");
        constexpr int32_t kMost = kForm == kUnits ? 3 << 20 : 1 << 30;
#pragma unroll
        for (int h = 0; h < WTN / 64; ++h) {
            const int nl = 64 * h + lane;
            const int32_t tv = thr_tab[nl];
            const uint32_t fv = flip_tab[nl];
            const int32_t tc = tv < -kMost ? -kMost : (tv > kMost ? kMost : tv);
            const int32_t e = (int32_t)((uint32_t)(tc - 1) - column_term(h) - mc.c0);
            if constexpr (kForm == kUnits)
                reinterpret_cast<float *>(thr_tab)[nl] = (float)e;
            else
                thr_tab[nl] = e;
            flip_tab[nl] = fv != 0 ? (1u << ((nl & 0x18) | (nl & 3))) : 0u;
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the wave's own LDS writes have landed
        __builtin_amdgcn_wave_barrier();
    } else if constexpr (kTerms == kBothTerms) {
        if (kg == 0) {
#pragma unroll
            for (int b = 0; b < WBN; ++b) {
                const uint32_t term = mc.cRW * (uint32_t)rw[b];
                if constexpr (kForm == kUnits)
                    reinterpret_cast<float *>(rw_tab)[b * 32 + r] = (float)(int32_t)(term + mc.c0) + kMagic;
                else
                    rw_tab[b * 32 + r] = term;
            }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_wave_barrier();
    }
    int64_t m_of[WB];
    uint32_t mterm[WB];
    float mterm_f[WB];
#pragma unroll
    for (int bj = 0; bj < WB; ++bj) {
        m_of[bj] = m_wave + bj * 32 + r;
        const uint32_t term = kTerms == kNoTerms ? 0u : mc.cRA * (uint32_t)ra[bj];
        mterm[bj] = kSign ? term : (kForm == kUnits ? term - kMagicBits : term + mc.c0);
        mterm_f[bj] = -(float)(int32_t)term;
    }
    // the product of the raw codes as it enters C
    auto scaled = [&](auto a) __attribute__((always_inline)) -> uint32_t {
        if constexpr (kForm == kShift)
            return acc_to_sum(a) << mc.alpha_shift;
        else
            return acc_to_sum(a) * mc.alpha;
    };
    // kInside, kLower int32 output: lines of the block before the current one, read from LDS and not stored yet; lane
    // (row = lane / 8, 16-byte unit = lane mod 8) of store j writes row 8 j + lane / 8 of the block
    i32x4 pend[4];
    int32_t *const line_base = kSign ? nullptr : g.epi.C + (m_wave + (lane >> 3)) * g.epi.ldc + n_wave + 4 * (lane & 7);
    auto store_lines = [&](const int pbi, const int pbj) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (kTile == kInside || m_wave + pbj * 32 + 8 * j + (lane >> 3) < g.M)
                *reinterpret_cast<i32x4 *>(line_base + (int64_t)(pbj * 32 + 8 * j) * g.epi.ldc + pbi * 32) = pend[j];
    };
    uint32_t word[WBN];  // thresholds: of row m_wave + lane
#pragma unroll
    for (int bi = 0; bi < WBN; ++bi) {
        const int64_t n_blk = n_wave + bi * 32;
        uint32_t nterm[16];  // int32 sums: the part that depends on n only
        if constexpr (!kSign && kTerms == kBothTerms) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint4 t4 = *reinterpret_cast<const uint4 *>(&rw_tab[bi * 32 + 8 * q + 4 * kg]);
                nterm[4 * q] = t4.x, nterm[4 * q + 1] = t4.y, nterm[4 * q + 2] = t4.z, nterm[4 * q + 3] = t4.w;
            }
        }
        if constexpr (!kSign) {
#pragma unroll
            for (int bj = 0; bj < WB; ++bj) {
                int32_t *row = g.epi.C + m_of[bj] * g.epi.ldc + n_blk + 4 * kg;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    i32x4 val;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (kForm == kUnits) {
                            static_assert(kTerms == kBothTerms, "the column table holds the float constant");
                            val[i] = (int32_t)(__float_as_uint(__builtin_fmaf(alpha, acc[bi][bj][4 * q + i], __uint_as_float(nterm[4 * q + i]))) + mterm[bj]);
                        } else if constexpr (kTerms == kBothTerms) {
                            val[i] = (int32_t)(scaled(acc[bi][bj][4 * q + i]) + nterm[4 * q + i] + mterm[bj]);
                        } else if constexpr (kTerms == kRowTerms) {
                            val[i] = (int32_t)(scaled(acc[bi][bj][4 * q + i]) + mterm[bj]);
                        } else {
                            val[i] = (int32_t)scaled(acc[bi][bj][4 * q + i]);
                        }
                    }
                    if constexpr (kFast || !kScatterEdge) {
                        // 16-byte unit 2 q + kg of row r, swizzled with the row: neither this write nor the read
                        // below puts two lanes of a pass on one LDS bank
                        *reinterpret_cast<i32x4 *>(&stage_w[r * 32 + 4 * ((2 * q + kg) ^ ((r >> 1) & 7))]) = val;
                    } else if (m_of[bj] < g.M) {
                        const int64_t n0 = n_blk + 8 * q + 4 * kg;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (n0 + i < g.N) row[8 * q + i] = val[i];
                    }
                }
                if constexpr (kFast) {
                    // read the block back as 8 rows x 128 bytes per instruction (LDS operations of a wave execute
                    // in order; only the compiler has to be kept from reordering them) and store those lines one
                    // block later, which hides the LDS round trip behind the next block's arithmetic
                    __builtin_amdgcn_wave_barrier();
                    i32x4 line[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int R = 8 * j + (lane >> 3);
                        line[j] = *reinterpret_cast<const i32x4 *>(&stage_w[R * 32 + 4 * ((lane & 7) ^ ((R >> 1) & 7))]);
                    }
                    __builtin_amdgcn_wave_barrier();
                    if (bi + bj > 0) store_lines((bi * WB + bj - 1) / WB, (bi * WB + bj - 1) % WB);
#pragma unroll
                    for (int j = 0; j < 4; ++j) pend[j] = line[j];
                } else if constexpr (!kScatterEdge) {
                    // the right edge of C, or rows of C at any alignment: two rows x 32 words per instruction (16 as before, but of 32
                    // rows x two words each; merged 4 x 4 bit planes, 2240 x 1001 x 999: 47.9 -> 34.7 us, 1000 x 4096 x 2048: 52.4 -> 47.3)
                    const int col = lane & 31;
                    const int32_t *const unit = stage_w + (lane & 3);
                    __builtin_amdgcn_wave_barrier();
                    int32_t word[16];
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const int R = 2 * j + kg;
                        word[j] = unit[R * 32 + 4 * ((col >> 2) ^ ((R >> 1) & 7))];
                    }
                    __builtin_amdgcn_wave_barrier();
                    const int64_t m_blk = m_wave + bj * 32;
                    if (n_blk + col < g.N) {
                        int32_t *const dst = g.epi.C + m_blk * g.epi.ldc + n_blk + col;
#pragma unroll
                        for (int j = 0; j < 16; ++j)
                            if (m_blk + 2 * j + kg < g.M) dst[(int64_t)(2 * j + kg) * g.epi.ldc] = word[j];
                    }
                }
            }
        } else {
            // e[v] = T - 1 - (part of C that depends on n only): C >= T  <=>  e[v] - (rest of C) < 0.  All terms
            // are below 2^30 in magnitude (the host checks the bound of C, thresholds are clamped to it, which
            // does not change any comparison), so the differences cannot wrap.
            int32_t e[16];
            uint32_t flips = 0;  // at the bit positions 8 (v / 4) + v mod 4 of the partial word
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = bi * 32 + 8 * q + 4 * kg;
                const int4 t4 = *reinterpret_cast<const int4 *>(&thr_tab[col]);
                const uint4 f4 = *reinterpret_cast<const uint4 *>(&flip_tab[col]);
                e[4 * q + 0] = t4.x, e[4 * q + 1] = t4.y, e[4 * q + 2] = t4.z, e[4 * q + 3] = t4.w;
                flips |= f4.x | f4.y | f4.z | f4.w;
            }
            uint32_t both[WB];
#pragma unroll
            for (int bj = 0; bj < WB; ++bj) {
                // four bits per group of consecutive n, most significant first: the sign bit of e[v] - (rest of
                // C) is appended with one funnel shift; flips are applied to the whole word
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t nib = 0;
#pragma unroll
                    for (int i = 3; i >= 0; --i) {
                        const int v = 4 * q + i;
                        uint32_t x;
                        if constexpr (kForm == kUnits)
                            x = __float_as_uint(__builtin_fmaf(-alpha, acc[bi][bj][v], __int_as_float(e[v]) + mterm_f[bj]));
                        else
                            x = (uint32_t)e[v] - (scaled(acc[bi][bj][v]) + mterm[bj]);
                        nib = __builtin_amdgcn_alignbit(nib, x, 31);  // (nib << 1) | (x >> 31)
                    }
                    bits |= nib << (8 * q);
                }
                both[bj] = or_halves((bits ^ flips) << (4 * kg));
            }
            static_assert(!kSign || WB == 2, "a lane keeps one row of 64");
            word[bi] = kg ? both[WB - 1] : both[0];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kFast && !kSign) store_lines(WBN - 1, WB - 1);
    if constexpr (kSign) store_words<WBN>(g, word, m_wave + lane, n_wave);
}

// Chooses the epilogue variant for a finished wave tile (interior or edge, form of C).  Tiles at the lower edge
// alone keep the whole-line stores: with the word stores of kAny they were the last to finish (256 x 128 tiles, 10000 x 512 x 2048:
// 16.4 -> 13.4 us, 1000 x 4096 x 2048 17.7 -> 14.1; merged 4 x 4 bit planes, 2240 x 4096 x 2048: 46.8 -> 43.8).  Not in the widest
// tile, whose registers are full.
template <bool kSign, int WBN, int kLoadsAfter, Terms kTerms, int WB, typename Acc>
__device__ __forceinline__ void wave_finish(const GemmArgs &g, const MfmaConst &mc, Acc (&acc)[WBN][WB], int32_t (&ra)[WB],
                                            int32_t (&rw)[WBN], uint32_t *rw_tab, int32_t *thr_tab, uint32_t *flip_tab,
                                            int32_t *stage_w, const int64_t m_wave, const int64_t n_wave) {
    const bool rows_inside = m_wave + 32 * WB <= g.M, columns_inside = n_wave + 32 * WBN <= g.N;
    const bool wide = kSign || ((g.epi.ldc % 4 == 0) && (reinterpret_cast<uintptr_t>(g.epi.C) % 16 == 0));
    auto finish = [&](auto form) __attribute__((always_inline)) {
        constexpr Form kForm = decltype(form)::value;
        if (wide && columns_inside && rows_inside) {
            wave_epilogue<kSign, WBN, kInside, kLoadsAfter, kTerms, kForm>(g, mc, acc, ra, rw, rw_tab, thr_tab, flip_tab, stage_w, m_wave, n_wave);
            return;
        }
        if constexpr (!kSign && WBN * WB < 16) {
            if (wide && columns_inside) {
                wave_epilogue<kSign, WBN, kLower, kLoadsAfter, kTerms, kForm>(g, mc, acc, ra, rw, rw_tab, thr_tab, flip_tab, stage_w, m_wave, n_wave);
                return;
            }
        }
        wave_epilogue<kSign, WBN, kAny, kLoadsAfter, kTerms, kForm>(g, mc, acc, ra, rw, rw_tab, thr_tab, flip_tab, stage_w, m_wave, n_wave);
    };
    constexpr bool kCanUnits = kTerms == kBothTerms && std::is_same_v<Acc, mfma::v16f> && WBN * WB < 16;
    if (kCanUnits ? mc.units != 0 : mc.alpha_shift >= 0)
        finish(std::integral_constant<Form, kCanUnits ? kUnits : kShift>{});
    else
        finish(std::integral_constant<Form, kTimes>{});
}

}  // namespace panel
}  // namespace qnn
