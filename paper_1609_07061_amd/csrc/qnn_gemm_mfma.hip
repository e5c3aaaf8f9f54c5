// Matrix-core engine of the binary / bit-plane matrix product: host side (operand codes, epilogue constants, choice of
// the kernel instantiation, launch).  The kernel itself is in qnn_gemm_mfma_kernel.h.

#include "qnn_gemm_mfma_kernel.h"
#include "qnn_gemm_bytes_panel_kernel.h"
#include "qnn_gemm_panel_kernel.h"
#include "qnn_gemm_stage_kernel.h"

namespace qnn {

using namespace mfma;

namespace {

// Derives the int8 code of one operand; false if its coefficients do not fit (then the vector-ALU engine is used).
bool make_code(const Planes &pl, Code &c, int64_t &alpha, int64_t &beta, int64_t &x_pad) {
    const int P = pl.count;
    int64_t gcd = 0;
    for (int p = 0; p < P; ++p) {
        int64_t a = pl.coef[p] < 0 ? -(int64_t)pl.coef[p] : pl.coef[p];
        if (a == 0) return false;
        int64_t x = gcd, y = a;
        while (y) {
            int64_t t = x % y;
            x = y;
            y = t;
        }
        gcd = x;
    }
    if (P == 1 && pl.coef[0] < 0) gcd = -gcd;  // a single plane keeps its bit as it is; the sign goes into alpha
    uint32_t used = 0;
    int64_t U = 0, neg = 0, sum_c = 0;
    for (int p = 0; p < P; ++p) {
        const int64_t d = pl.coef[p] / gcd;
        const int64_t ad = d < 0 ? -d : d;
        if (ad > 128 || (ad & (ad - 1)) != 0) return false;  // power of two up to 128
        int lg = 0;
        while ((1 << lg) < ad) ++lg;
        if (used & (1u << lg)) return false;  // positions must be distinct for the OR
        used |= 1u << lg;
        c.lg[p] = lg;
        c.inv[p] = d < 0 ? 0xFFFFFFFFu : 0u;
        c.d[p] = (int32_t)d;
        U += ad;
        if (d < 0) neg += ad;
        sum_c += pl.coef[p];
    }
    for (int p = P; p < QNN_MAX_PLANES; ++p) c.lg[p] = 0, c.inv[p] = 0, c.d[p] = 0;
    const int64_t offp = U > 127 ? 128 : 0;
    c.bias = offp ? 0x80808080u : 0u;
    const int64_t off = offp - neg;  // x8 = sum_p d_p b_p - off
    if (pl.mode == QNN_PLANE_BIT) {
        alpha = gcd;
        beta = gcd * off;
    } else {
        alpha = 2 * gcd;
        beta = 2 * gcd * off - sum_c;
    }
    x_pad = -off;
    return true;
}


// Epilogue constants of C = aA aW (S - npad xA0 xW0) + aA bW RA[m] + bA aW RW[n] + K bA bW for a kernel that processes
// Kproc >= K elements per row (the surplus reads as zero bits); false if the sums could leave the exact range.
bool fill_consts(const GemmArgs &g, int64_t aA, int64_t bA, int64_t xA0, int64_t aW, int64_t bW, int64_t xW0,
                 int64_t Kproc, MfmaConst &mc) {
    if (g.epi.T) {
        // the threshold epilogue compares through differences, which must not wrap: |C| < 2^30
        long double bound = (long double)g.K;
        long double sa = 0, sw = 0;
        for (int p = 0; p < g.pa.count; ++p) sa += g.pa.coef[p] < 0 ? -(long double)g.pa.coef[p] : g.pa.coef[p];
        for (int p = 0; p < g.pw.count; ++p) sw += g.pw.coef[p] < 0 ? -(long double)g.pw.coef[p] : g.pw.coef[p];
        if (bound * sa * sw >= 1073741824.0L) return false;
    }
    if (Kproc >= 131072) return false;  // |S| <= Kproc * 2^14 must stay below 2^31
    const int64_t npad = Kproc - g.K;
    mc.msteps = 0;
    mc.alpha = (uint32_t)(aA * aW);
    mc.cRA = (uint32_t)(aA * bW);
    mc.cRW = (uint32_t)(bA * aW);
    mc.c0 = (uint32_t)(g.K * bA * bW - aA * aW * npad * xA0 * xW0);
    mc.needRW = mc.cRW != 0;
    auto unit = [](const Planes &pl) { return pl.count == 1 && (pl.coef[0] == 1 || pl.coef[0] == -1); };
    mc.units = !g.A.rows_are_bytes && unit(g.pa) && unit(g.pw);
    // the row sums are over the true K: RA = sum_p d_p pop_p - K * off; fold the constant part into c0
    mc.c0 += (uint32_t)(aA * bW * (g.K * xA0)) + (uint32_t)(bA * aW * (g.K * xW0));
    mc.alpha_shift = -1;
    for (int sh = 0; sh < 31; ++sh)
        if (aA * aW == ((int64_t)1 << sh)) mc.alpha_shift = sh;
    return true;
}

const Variant *find_variant(const GemmArgs &g) {
    const bool pixels = g.A.rows_are_pixels != 0, sign = g.epi.T != nullptr;
    const VariantList lists[] = {variants_fp4(), variants_first_layer(), variants_multibit(), variants_conv(),
                                   variants_conv_sign()};
    for (const VariantList &l : lists)
        for (int i = 0; i < l.n; ++i) {
            const Variant &v = l.v[i];
            if (v.PA == g.pa.count && v.PW == g.pw.count && v.pixels == pixels && v.sign == sign) return &v;
        }
    return nullptr;
}

bool prepare(const GemmArgs &g, bool fp4, const Variant *&var, MfmaConst &mc, bool &vec) {
    static const Variant kBytes = {0, 1, 1, false, false, nullptr, nullptr, nullptr, nullptr};
    const bool bytes = g.A.rows_are_bytes != 0;
    int64_t aA, bA, xA0, aW, bW, xW0;
    if (bytes) {
        // x8 = code - 128, true value = x8 + 128; rows of 16-byte aligned chunks only
        if (fp4 || g.pw.count != 1 || g.K % 16 || g.A.ld % 16 || reinterpret_cast<uintptr_t>(g.A.base) % 16) return false;
        var = &kBytes;
        std::memset(&mc.a, 0, sizeof(mc.a));
        aA = 1, bA = 128, xA0 = 0;
        if (!make_code(g.pw, mc.w, aW, bW, xW0)) return false;
    } else {
        var = find_variant(g);
        if (!var) return false;
        if (fp4 && !var->fp4_vec) return false;
        if (!make_code(g.pa, mc.a, aA, bA, xA0) || !make_code(g.pw, mc.w, aW, bW, xW0)) return false;
    }
    const int64_t step_words = 2 * var->WPL;
    const int64_t msteps = 2 * ceil_div(g.Kw, 2 * step_words);
    if (!fill_consts(g, aA, bA, xA0, aW, bW, xW0, msteps * step_words * 32, mc)) return false;
    mc.msteps = (uint32_t)msteps;
    // vector loads need every row (of every plane) to start at a multiple of the load width and to be made of whole
    // chunks, so that a chunk is either all inside or all outside the row
    const int wpl = var->WPL;
    auto aligned = [&](const uint32_t *base, int64_t ld, int64_t pstride, int planes) __attribute__((always_inline)) {
        if (reinterpret_cast<uintptr_t>(base) % (4 * wpl)) return false;
        if (planes > 1 && pstride % wpl) return false;
        return ld % wpl == 0;
    };
    const bool pix = g.A.rows_are_pixels != 0;
    vec = !bytes && wpl > 1 && aligned(g.A.base, pix ? g.A.Cw : g.A.ld, g.A.plane_stride, g.pa.count) &&
          aligned(g.W, g.ldw, g.strideW, g.pw.count) && (pix ? g.A.Cw % wpl == 0 : true) && g.Kw % wpl == 0;
    return true;
}

}  // namespace

bool mfma_supports(const GemmArgs &g, bool fp4) {
    const Variant *v;
    MfmaConst mc;
    bool vec;
    return prepare(g, fp4, v, mc, vec);
}

bool mfma_preferred(const GemmArgs &g) {
    // small or skinny products (a 10-neuron output layer fills 10 of a tile's 256 columns) are better served by the
    // finer tiles of the vector-ALU engine
    if (ceil_div(g.M, BM) * ceil_div(g.N, BN) >= 32 && g.K >= 256 && g.M >= 128 && g.N >= 128) return true;
    // single planes with long rows: a few matrix-core tiles beat many vector-ALU tiles (a fully connected layer of 8192
    // inputs on a batch of 256: 27 us on eight 256 x 128 tiles against 41 us on sixty-four 64 x 64 tiles)
    return g.pa.count == 1 && g.pw.count == 1 && !g.A.rows_are_pixels && !g.A.rows_are_bytes && g.K >= 4096 && g.M >= 256 &&
           g.N >= 256;
}

int compute_units() {
    static thread_local int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cus = n;
    }
    return cus;
}

// Tiles of the byte-operand kernel: 64 `blocks` rows x 256 columns, taken in rounds of one tile per compute unit.  In units of a
// round of 128 rows, rounds of 256 and 192 rows cost 1.41 and 1.22 (reads of LDS and matrix cores overlap worse the fewer products
// an operand feeds; per group of k, random operands: 0.94, 1.23 and 1.30 us with 128, 192, 256 rows), and one of halved 256-row tiles,
// possible where the last round has tiles for at most half of the compute units, 1.03; the fewest rounds by that cost are taken.  (The
// measured costs would take halves where 192 rows are faster: 7757 x 4231 x 4096, 179 us against 169.)  With 256 rows -> as chosen,
// merge of 4 x 4 planes included: 2240 x 4096 x 2048 (144 -> 192 tiles) 45.5 -> 43.6 us, x 4096 64.3 -> 59.2; 1000 x 4096 x 4096 (64 ->
// 128) 58.7 -> 44.9; 2000 x 3000 x 1500 (96 -> 192) 39.8 -> 32.0; 10000 x 4096 x 4096 keeps 2.5 rounds of 256 rows.
struct BytesTiles {
    int blocks;
    bool tail;
    int64_t tiles_m, tiles_n;
    unsigned grid;
    double rounds;  // by that cost
};
static BytesTiles bytes_tiles(int64_t M, int64_t N, int cus) {
    constexpr double kRound[5] = {0.0, 0.0, 1.0, 1.22, 1.41}, kHalves = 1.03;
    BytesTiles t = {4, false, 0, ceil_div(N, 256), 0, 0.0};
    for (int blocks = 4; blocks >= 2; --blocks) {
        const int64_t tiles_m = ceil_div(M, 64 * blocks), total = tiles_m * t.tiles_n, whole = total / cus, rest = total % cus;
        const bool tail = blocks == 4 && cus % 16 == 0 && whole > 0 && rest != 0 && 2 * rest <= cus;
        const double cost = kRound[blocks] * (double)whole + (tail ? kHalves : (rest ? kRound[blocks] : 0.0));
        if (blocks == 4 || cost < t.rounds) t.blocks = blocks, t.tail = tail, t.tiles_m = tiles_m, t.grid = (unsigned)(total < cus ? total : cus), t.rounds = cost;
    }
    return t;
}

// What the panel-fed kernels take: single planes of matrices that span less than 4 GiB with a tile beyond the last row (row offsets are
// 32-bit, and the wide kernel forms them before it clamps them).
static bool panel_layout(const GemmArgs &g) {
    const bool spans32 = 4.0L * (long double)(g.M + 256) * g.A.ld < 4294967296.0L && 4.0L * (long double)(g.N + 256) * g.ldw < 4294967296.0L;
    return spans32 && g.pa.count == 1 && g.pw.count == 1 && !g.A.rows_are_pixels && !g.A.rows_are_bytes;
}

// Which of the panel-fed kernels and tiles: by the time of their rounds (us; k = thousands of 1024 elements).  Tiles of 128 x 256, 256 x 128
// or 128 x 128, two workgroups on a compute unit (three with 128 x 128 and thresholds, whose registers allow it: first 128-filter
// convolution of the App. A network on 256 images, 2048 tiles, 30.8 -> 26.1): a round with two and with one on a unit; a thinly filled last round
// and the padding of a ragged edge both show.  (128 x 256 -> 128 x 128: 10000 x 4096 x 4096 with thresholds 55.7 and 64.2, 3000 x 4096 x
// 4096 24.2 and 19.3, 10000 x 2048 x 2048 21.5 and 19.6, 262144 x 128 x 1024 36.9 and 21.9, 700 x 4096 x 4096 15.8 and 10.5; before, on 256
// x 256 and 256 x 128 tiles of one workgroup, 60.3, 24.9, 26.1, 24.4, 14.7.)  Int32 sums on 256 x 256 tiles of one workgroup where
// that costs less: rounds of 9.5 + 4.1 k against 8.2 + 4.55 k.
struct PanelTiles {
    panel::Shape shape;
    int per;    // workgroups on a compute unit
    bool wide;  // 256 x 256, one workgroup
    PanelTiles(int64_t M, int64_t N, int64_t Kw, bool sign, bool map, int64_t cus) {
        const double k = (double)Kw / 32.0;
        // (a last round of few tiles runs at a higher clock: 6144^3, two rounds and 128 tiles of 128 x 256, 81.8, of 128 x 128 88.7)
        auto rounds = [cus](int64_t tiles, double two, double one) {
            const int64_t whole = tiles / (2 * cus), rest = tiles % (2 * cus);
            const double last = rest > cus ? two : (whole > 0 ? (0.4 + 0.6 * (double)rest / (double)cus) * one : one);
            return (double)whole * two + (rest == 0 ? 0.0 : last);
        };
        const int64_t tm = ceil_div(M, 128), tn = ceil_div(N, 128);
        const double end = sign ? (map ? 3.0 : 0.0) : 4.7;  // what the epilogue takes beyond that of plain thresholds
        const double two = 3.5 + end + 4.55 * k, one = 2.2 + 0.7 * end + 2.55 * k;
        const double large = rounds(tm * ceil_div(N, 256), two, one), tall = rounds(ceil_div(M, 256) * tn, two, one);
        const double small = rounds(tm * tn, 2.2 + (map ? 0.5 : 0.6 * end) + 2.4 * k, 1.2 + (map ? 0.3 : 0.4 * end) + 1.6 * k);
        const double best = large <= tall ? large : tall;
        shape = small < 0.98 * best ? panel::k128x128 : (large <= tall ? panel::k128x256 : panel::k256x128);
        per = shape == panel::k128x128 && sign ? 3 : 2;
        wide = !sign && Kw % panel::kWideGroupWords == 0 && (double)ceil_div(ceil_div(M, 256) * ceil_div(N, 256), cus) * (9.5 + 4.125 * k) < (small < 0.98 * best ? small : best);
    }
};

void panel_shape(int64_t M, int64_t N, int64_t Kw, int &shape, int &per) {
    const PanelTiles t(M, N, Kw, true, true, compute_units());
    shape = t.shape, per = t.per;
}

bool panel_takes(const GemmArgs &g) {
    const Variant *v;
    MfmaConst mc;
    bool vec;
    return g.K >= 512 && prepare(g, true, v, mc, vec) && panel_layout(g);
}

int launch_gemm_mfma(const GemmArgs &g, hipStream_t s, bool fp4) {
    const Variant *v;
    MfmaConst mc;
    bool vec;
    if (!prepare(g, fp4, v, mc, vec)) return fail(QNN_ERR_UNSUPPORTED, "matrix-core engine cannot take these arguments");
    const int64_t tiles_m = ceil_div(g.M, BM), tiles_n = ceil_div(g.N, BN);
    if (tiles_m * tiles_n > 0x7FFFFFFFLL) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
    // one persistent workgroup per compute unit (each takes 512 registers per lane, so one fits)
    const int cus = compute_units();
    const int64_t total = tiles_m * tiles_n;
    const unsigned grid = (unsigned)(total < cus ? total : cus);
    // single-plane products on the FP4 path: the panel-fed kernels
    if (fp4 && panel_layout(g)) {
        const bool whole = vec && g.Kw % panel::kGroupWords == 0;
        int64_t aA, bA, xA0, aW, bW, xW0;
        MfmaConst pc = mc;
        panel::PanelArgs pa;
        std::memset(&pa, 0, sizeof(pa));
        pa.steps = (uint32_t)(whole ? g.Kw / 8 : ceil_div(g.Kw, 8));
        if (make_code(g.pa, pc.a, aA, bA, xA0) && make_code(g.pw, pc.w, aW, bW, xW0) &&
            fill_consts(g, aA, bA, xA0, aW, bW, xW0, (int64_t)pa.steps * 256, pc)) {
            const PanelTiles pt(g.M, g.N, g.Kw, g.epi.T != nullptr, false, cus);
            if (pt.wide && whole) {
                const unsigned wgrid = (unsigned)(total < cus ? total : cus);
                return QNN_LAUNCH("gemm_panel_wide", panel::wide_kernel(), dim3(wgrid), dim3(panel::kThreads), 0, s, g, pc, (uint32_t)tiles_m, (uint32_t)tiles_n,
                                  (uint32_t)(g.Kw / panel::kWideGroupWords));
            }
            const int64_t pm = ceil_div(g.M, panel::rows_of(pt.shape)), pn = ceil_div(g.N, panel::columns_of(pt.shape)), per = pt.per * cus;
            if (pm * pn > 0x7FFFFFFFLL) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
            pa.tiles = make_tiles(pm, pn);
            pa.a_bytes = (uint32_t)(((g.M - 1) * g.A.ld + g.Kw) * 4), pa.w_bytes = (uint32_t)(((g.N - 1) * g.ldw + g.Kw) * 4);
            const unsigned pgrid = (unsigned)(pm * pn < per ? pm * pn : per);
            return QNN_LAUNCH("gemm_panel", panel::find_kernel(g.epi.T != nullptr, pt.shape, whole), dim3(pgrid), dim3(panel::kThreads), 0, s, g, pc, pa);
        }
    }
    if (codes::supports(g)) return codes::launch(g, s);
    const KernelFn fn = g.A.rows_are_bytes ? byte_kernels()[g.epi.T ? 1 : 0]
                        : fp4              ? (vec ? v->fp4_vec : v->fp4_any)
                                           : (vec ? v->fn_vec : v->fn_any);
    return QNN_LAUNCH("gemm_mfma", fn, dim3(grid), dim3(kThreads), 0, s, g, mc, (uint32_t)tiles_m,
                       (uint32_t)tiles_n);
}

// ------------------------------------------------------------------------------------------------ staged kernels
namespace {

using stage::StageConst;
typedef void (*StageFn)(const GemmArgs, const MfmaConst, const StageConst, uint32_t, uint32_t);

// One operand for the merge network: bit position q of the code comes from plane order[q]; false if the positions
// are not exactly 0 .. P-1 or the plane count has no network.
bool stage_operand(const Planes &pl, const Code &c, int64_t plane_stride, int64_t (&off)[QNN_MAX_PLANES],
                   uint32_t (&inv)[QNN_MAX_PLANES], int32_t (&d)[QNN_MAX_PLANES]) {
    const int P = pl.count;
    if (P != 1 && P != 2 && P != 4 && P != 8) return false;
    for (int q = 0; q < QNN_MAX_PLANES; ++q) off[q] = 0, inv[q] = 0, d[q] = 0;
    uint32_t seen = 0;
    for (int p = 0; p < P; ++p) {
        const int q = c.lg[p];
        if (q < 0 || q >= P || (seen & (1u << q))) return false;
        seen |= 1u << q;
        off[q] = (int64_t)p * plane_stride;
        inv[q] = c.inv[p];
        d[q] = c.d[p];
    }
    return true;
}

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

bool prepare_stage(const GemmArgs &g, MfmaConst &mc, StageConst &sc, StageFn &fn) {
    const bool pix = g.A.rows_are_pixels != 0, sign = g.epi.T != nullptr;
    if (g.A.rows_are_bytes) return false;
    std::memset(&sc, 0, sizeof(sc));
    int64_t aA, bA, xA0, aW, bW, xW0;
    if (!make_code(g.pa, mc.a, aA, bA, xA0) || !make_code(g.pw, mc.w, aW, bW, xW0)) return false;
    if (!stage_operand(g.pa, mc.a, g.A.plane_stride, sc.offA, sc.invA, sc.dA)) return false;
    if (!stage_operand(g.pw, mc.w, g.strideW, sc.offW, sc.invW, sc.dW)) return false;
    sc.biasA = mc.a.bias, sc.biasW = mc.w.bias;
    // 16-byte loads: every row of every plane starts on a 16-byte boundary and holds whole groups of four words
    const bool w_vec = aligned16(g.W) && g.ldw % 4 == 0 && (g.pw.count == 1 || g.strideW % 4 == 0) && g.Kw % 4 == 0;
    const bool a_vec = aligned16(g.A.base) && (g.pa.count == 1 || g.A.plane_stride % 4 == 0) &&
                       (pix ? g.A.Cw % 4 == 0 : (g.A.ld % 4 == 0 && g.Kw % 4 == 0));
    if (!a_vec || !w_vec) return false;
    // the kernel addresses rows with 32-bit offsets from a plane's base
    const long double a_span = pix ? 4.0L * (long double)g.M / ((long double)g.A.Ho * g.A.Wo) * g.A.H * g.A.Wd * g.A.Cw
                                   : 4.0L * (long double)g.M * g.A.ld;
    if (a_span >= 4294967296.0L || 4.0L * (long double)g.N * g.ldw >= 4294967296.0L) return false;
    const int64_t nmacro = ceil_div(g.Kw, 4);
    sc.nmacro = (uint32_t)nmacro;
    if (!fill_consts(g, aA, bA, xA0, aW, bW, xW0, nmacro * 4 * 32, mc)) return false;
    fn = stage::find_kernel(g.pa.count, g.pw.count, pix ? stage::kPixelPlanes : stage::kPlanes, sign);
    return fn != nullptr;
}

// Large products of multi-plane operands with int32 output: the planes of both operands are merged to int8 values once
// per call, into memory borrowed from the stream's pool, and the panel-fed byte kernel multiplies them.  (Merging in
// every workgroup repeats the work for every tile of a row of tiles and holds the multiplication up behind loads of
// one row per lane.)
// Row pitch of the merged operands: whole groups of k.
int64_t values_pitch(int64_t K) {
    const int64_t p = ceil_div(K, bytes_panel::kGroupK) * bytes_panel::kGroupK;
    return p;
}
bool values_path(const GemmArgs &g) {
    if (g.A.rows_are_pixels || g.A.rows_are_bytes || g.epi.T) return false;
    if (g.pa.count == 1 && g.pw.count == 1) return false;
    if (g.K < 512 || g.K >= 131072 || g.M < 256 || g.N < 256) return false;  // |S| <= K 2^14 stays below 2^31
    if ((long double)g.M * (long double)g.N * (long double)g.K < 2147483648.0L) return false;  // small: not worth three launches
    const int64_t pitch = values_pitch(g.K);
    if ((long double)(g.M + 256) * pitch >= 4294967296.0L || (long double)(g.N + 256) * pitch >= 4294967296.0L) return false;
    if (ceil_div(g.M, 256) * ceil_div(g.N, 128) > 0x7FFFFFFFLL) return false;
    return bytes_panel::merge_supports(g.pa, g.pw);
}

// C = alpha S of two operands of int8 values, rows of `pitch` bytes
int launch_values_product(const GemmArgs &g, const int8_t *a8, const int8_t *w8, int64_t pitch, int64_t alpha, hipStream_t s) {
    GemmArgs v = g;
    v.A.base = reinterpret_cast<const uint32_t *>(a8);
    v.A.ld = pitch;
    v.A.plane_stride = 0;
    v.A.rows_are_bytes = 1;
    v.w_bytes = w8;
    v.ld_w_bytes = pitch;
    MfmaConst mc;
    std::memset(&mc, 0, sizeof(mc));
    mc.alpha = (uint32_t)alpha;
    mc.alpha_shift = -1;
    for (int sh = 0; sh < 31; ++sh)
        if (alpha == ((int64_t)1 << sh)) mc.alpha_shift = sh;
    const BytesTiles bt = bytes_tiles(g.M, g.N, compute_units());
    return QNN_LAUNCH("gemm_values", bytes_panel::kernel_values(bt.tail, bt.blocks), dim3(bt.grid), dim3(bytes_panel::kThreads), 0, s, v, mc,
                      (uint32_t)bt.tiles_m, (uint32_t)bt.tiles_n, (uint32_t)ceil_div(g.K, bytes_panel::kGroupK));
}

int launch_values(const GemmArgs &g, hipStream_t s) {
    const int64_t pitch = values_pitch(g.K);
    const size_t bytes_a = (size_t)g.M * (size_t)pitch, bytes_w = (size_t)g.N * (size_t)pitch;
    PoolMemory mem(s);
    if (int rc = mem.take(bytes_a + bytes_w)) return rc;
    int8_t *a8 = static_cast<int8_t *>(mem.ptr), *w8 = a8 + bytes_a;  // (bytes_a is a multiple of 128)
    int64_t scale = 0;
    int rc = bytes_panel::launch_merge_planes(g, a8, w8, pitch, scale, s);
    if (rc == QNN_OK) rc = launch_values_product(g, a8, w8, pitch, scale, s);
    return mem.give_back(rc);
}

// One product of the backward step as a bit-plane product (for the choice of the way it takes).
GemmArgs backward_product(const BackwardArgs &b, int64_t M, int64_t N, int64_t K, int32_t *C, int64_t ldc) {
    GemmArgs g;
    std::memset(&g, 0, sizeof(g));
    g.pa = b.pg;
    g.pw.count = 1, g.pw.mode = QNN_PLANE_SIGN, g.pw.coef[0] = 1;
    g.A.base = b.G, g.W = b.W;
    g.M = M, g.N = N, g.K = K, g.Kw = words_for(K);
    g.A.ld = g.ldw = g.Kw;
    g.epi.C = C, g.epi.ldc = ldc;
    return g;
}

}  // namespace

// Whether the step takes the way of qnn_gemm_mixed.hip (FP6 or int8 gradients) or products of bit planes behind bit transposes.
//   More than four planes: by the expected times, with int8 gradients, the slower ones, and only where those of the planes, which the
//   estimates of the products undershoot, are 10 % higher (us behind the quantizer, planes -> FP6 / int8; eight planes: 10000 x 4096 x 4096 356 ->
//   220 / 340; 1009 x 1280 x 2784 62 -> 39; 7572 x 2368 x 444 158 -> 72 / 90; 1718 x 452 x 1895 55 -> 42 / 45; six planes: 3031 x 2083 x 906 82 ->
//   51 / 60).  Where a product has few tiles and long rows, the planes' kernels split k and this way's do not (10000 x 300 x 300 58 against 60 /
//   82, 20000 x 100 x 1000 90 against 100 / 139, 393 x 3517 x 960 44 against 43 / 48, all left to the planes).  A gradient that turns out int8
//   can lose where 128 x 256 tiles make between one and two rounds (7708 x 7094 x 1521, five planes, 221 -> 177 / 255).
//   Up to four planes, which make two pairs of digits at most: where merging them to bytes for each product would be faster than the
//   tiled kernel (a line that leaves steps to the planes which are faster here: 3000 x 2048 x 2048 with four planes 79 against 54).
bool backward_mixed_preferred(const BackwardArgs &b) {
    if (!mixed::backward_supports(b)) return false;
    const GemmArgs ga = backward_product(b, b.M, b.K, b.N, b.gA, b.ld_ga), gw = backward_product(b, b.N, b.K, b.M, b.gW, b.ld_gw);
    // (the transposes: three launches, two bits of traffic per bit at 2 TB/s)
    const double digits = 9.0 + 0.125e-6 * ((double)b.pg.count * b.M * b.N + (double)b.N * b.K + (double)b.M * b.K) + slice_us(ga) + slice_us(gw);
    if (b.pg.count > 4 && digits < 1e9) return mixed::backward_us(b) <= 1.1 * digits;
    double merged = 0.0;
    for (const GemmArgs *g : {&ga, &gw}) {
        if (!mfma_preferred(*g) || !values_path(*g)) return false;
        merged += stage_us(*g);
    }
    return merged <= digits;
}

// Merged once per call: products of 300 x 300 to 128000 x 256 rows and 512 to 30000 elements of k within 10 % as a rule (merge of both
// operands, groups of k by the tiles' rounds, store of C); merged per workgroup: rounds of 256 x 256 tiles (8192^3 of eight planes 881 us,
// 10000 x 4096 x 4096 361, 8192 x 8192 x 1024 197).
double stage_us(const GemmArgs &g) {
    const double elements = (double)g.M * (double)g.N;
    if (values_path(g))
        return 13.0 + 0.87 * bytes_tiles(g.M, g.N, compute_units()).rounds * (double)ceil_div(g.K, bytes_panel::kGroupK) + 0.85e-6 * elements +
               0.32e-6 * (double)(g.M + g.N) * (double)g.K;
    return 5.0 + 25e-3 * (double)ceil_div(ceil_div(g.M, 256) * ceil_div(g.N, 256), compute_units()) * (double)g.K + 0.8e-6 * elements;
}

bool stage_supports(const GemmArgs &g) {
    if (values_path(g)) return true;
    MfmaConst mc;
    StageConst sc;
    StageFn fn;
    return prepare_stage(g, mc, sc, fn);
}

int launch_gemm_stage(const GemmArgs &g, hipStream_t s) {
    if (values_path(g)) return launch_values(g, s);
    MfmaConst mc;
    StageConst sc;
    StageFn fn;
    if (!prepare_stage(g, mc, sc, fn))
        return fail(QNN_ERR_UNSUPPORTED, "staged matrix-core kernels cannot take these arguments");
    const int64_t tiles_m = ceil_div(g.M, 256), tiles_n = ceil_div(g.N, 256);
    if (tiles_m * tiles_n > 0x7FFFFFFFLL) return fail(QNN_ERR_SHAPE, "gemm: too many tiles");
    const int64_t total = tiles_m * tiles_n;
    const int cus = compute_units();
    const unsigned grid = (unsigned)(total < cus ? total : cus);
    return QNN_LAUNCH("gemm_stage", fn, dim3(grid), dim3(stage::kThreads), 0, s, g, mc, sc, (uint32_t)tiles_m,
                      (uint32_t)tiles_n);
}

}  // namespace qnn
