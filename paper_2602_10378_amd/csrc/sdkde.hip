// SD-KDE hot path for MI355X (gfx950 / CDNA4): prep, pair-interaction kernels (MFMA for d >= 4, direct
// differences for thin d), split reduction + epilogues, and the C ABI.
//
// Notation follows the paper: c = 1/(2h^2), phi_ij = exp(-c |p_i - x_j|^2),
// D_i = sum_j phi_ij, T_i = sum_j phi_ij x_j  (Method section: T = Phi X).
//
// All coordinates are taken relative to a centre of the samples and scaled by a = sqrt(c log2 e), so that
// the squared distance in scaled units is directly the (negated) argument of exp2:
//     phi_ij = exp2( 2 p~_i . x~_j - |p~_i|^2 - |x~_j|^2 ).
// The cross term is the Gram-matrix tile of the Method section, computed with MFMAs (fp32 operands as
// two fp16 parts each, half2.h); the score numerator uses Phi X with the Phi tile still in the
// registers the first MFMA left it in.
#include <string.h>
#include <atomic>
#include <mutex>
#include "common.h"
#include "prep.h"
#include "pair_mfma.h"
#include "pair_half.h"
#include "pair_whole.h"
#include "pair_split.h"
#include "pair_sym.h"
#include "pair_thin.h"
#include "epilogue.h"
#include "epilogue_prep.h"

namespace {

// ------------------------------------------------------------------------------------------
// Host side: plan, workspace layout, dispatch.
// ------------------------------------------------------------------------------------------

// Most row tiles per wave for which pair_mfma_kernel (fp16 input modes) is instantiated (larger ones would spill registers).
constexpr int max_row_tiles(int kb, int kind, int prec)
{
    if ((prec == SDKDE_PREC_FP16X2_ALL || prec == SDKDE_PREC_FP16X2_PHI16) && kb > 1) return 0;      // see effective_prec()
    const bool second = kind == kScoreSelf || kind == kScorePoints;       // has the Phi X contraction
    return second ? (kb == 1 ? 8 : kb <= 4 ? 4 : 2)
                  : (kb == 1 ? 16 : kb == 2 ? 8 : kb <= 4 ? 4 : 2);
}

// Shapes of pair_half_kernel: a workgroup of `waves` waves of `ni` row tiles each holds 16 ni waves rows; the plan counts
// them as rt = ni waves / 4 (so that a workgroup has 64 rt rows, as in the other kernels).  nb, ahead, minw: see there.
// ni = 0: not built.
// Clocks of a wave's 16 x 16 pairs (as in pair_half.h) with rt = 2 / 4 / 8: score d = 16 187 / 180 / 178; eval d = 16 83 / 77 / 75.
// Four row tiles a wave take the fewest operand reads that the registers allow up to dp = 32 (eval 96); above, eight waves of
// two share a workgroup's reads instead.  The score at dp = 48 has four at the samples themselves only, without reading ahead
// (both together spill), likewise four instead of eight at dp = 16 where sums are shifted.  Shifted sums need a few registers more:
// eval the Gram accumulators of two row tiles at a time instead of four at dp = 16 and two waves a SIMD at dp = 48, the score at
// d = 81 .. 88 one wave a SIMD in the smallest shape.
struct HalfShape { int ni, waves, nb; bool ahead; int minw; };
constexpr HalfShape half_shape(int kb, bool score, int rt, bool self = true, bool far = false, int tail = kTailSixteen)
{
    if (score) {
        if (rt == 2) return {2, 4, 2, true, kb == 1 && !far ? 4 : kb <= 2 ? 3 : kb <= 6 && !(far && kb == 6 && tail == kTailSpare) ? 2 : 1};
        if (rt == 4) return kb <= 2 ? HalfShape{4, 4, 4, true, 2} : kb == 3 && self ? HalfShape{4, 4, 2, false, 2} : kb <= 6 ? HalfShape{2, 8, 2, true, 2} : HalfShape{};
        if (rt == 8 && kb == 1) return far ? HalfShape{4, 8, 2, true, 2} : HalfShape{8, 4, 2, true, 2};
    } else {
        if (rt == 2) return {2, 4, 2, false, kb <= 2 ? 4 : kb <= 4 ? 3 : 2};
        if (rt == 4) return kb <= 6 ? HalfShape{4, 4, kb <= 3 && !(far && kb == 1) ? 4 : 2, false, kb <= (far ? 2 : 3) ? 3 : 2} : HalfShape{2, 8, 2, false, 2};
        if (rt == 8 && kb == 1) return {8, 4, 4, false, 2};
    }
    return {};
}
constexpr int max_half_rt(int kb, bool score)
{
    return half_shape(kb, score, 8).ni ? 8 : half_shape(kb, score, 4).ni ? 4 : 2;
}

// Precision mode a call actually runs in: the thin path is fp32 VALU code; the fp16 second contraction is
// used at dp = 16 only and falls back to fp16x2 above.  (Its split of Phi is VALU work that eight row tiles per
// wave amortise best, and from dp = 32 on only four fit: measured at n = 131072, fp16x2 against fp16x2-all,
// d = 32 10.7 / 11.3 ms and d = 64 21.7 / 22.3 ms, where d = 16 gives 6.0 / 4.4 ms.)
inline uint32_t effective_prec(uint32_t flags, bool thin, int dp)
{
    const uint32_t prec = flags & 15u;
    if (thin) return SDKDE_PREC_FP32;
    if ((prec == SDKDE_PREC_FP16X2_ALL || prec == SDKDE_PREC_FP16X2_PHI16) && dp > 16) return SDKDE_PREC_FP16X2;
    return prec;
}

// The fp16 split of 2^14 phi resolves weights with ABSOLUTE precision 2^-39 (the fp16 subnormal step over the
// scale), which is harmless next to a weight of one: the sample's own term at the samples themselves, the
// largest term after a max shift.  A score at separate points without that shift has no such anchor (a point
// whose weights are all below ~1e-7 would lose them in T but not in D), so it runs the fp16x2 mode instead.
inline uint32_t anchored_flags(uint32_t flags, bool self)
{
    const uint32_t prec = flags & 15u;
    if ((prec == SDKDE_PREC_FP16X2_ALL || prec == SDKDE_PREC_FP16X2_PHI16) && !self && !(flags & SDKDE_FLAG_MAX_SHIFT))
        return (flags & ~15u) | SDKDE_PREC_FP16X2;
    return flags;
}

struct Plan {
    bool thin;
    bool parts;           // the fp32 mode's matrix path: operands in parts, 6 bytes a value (pair_half_kernel; symmetric mode)
    int d, dp;            // true and padded dimension (thin: dp == d)
    int ni;               // MFMA: row tiles per wave; thin: rows per thread
    int rows_per_block;
    int64_t n_pad, m_pad; // padded sample / point row counts
    int ntiles;           // 16-sample tiles
    int nsplit, tiles_per_split;
    int64_t row_blocks;
    // symmetric mode of the score at the samples themselves (pair_sym_kernel), off unless sym_on
    bool sym_on;
    int sym_ni, sym_rb, sym_per_group, sym_nblocks, sym_ngroups;
};

// How a call's prepared rows are held (common.h), and the scale of its coordinates: sqrt(c log2 e),
// times sqrt 2 in the fp32 mode's formats, which carry the factor 2 of the cross term in both of their operands.
inline int operand_format(const Plan& p, uint32_t flags)
{
    return p.parts ? (p.sym_on ? kFormatSplit3 : kFormatHalf2) : (int)effective_prec(flags, p.thin, p.dp);
}
inline double operand_scale(int format, double h)
{
    return sqrt(1.4426950408889634074 / (format == kFormatSplit3 || format == kFormatHalf2 ? h * h : 2.0 * h * h));
}

// Overrides of the plan's own choices, set through sdkde_set_tuning (tests and sweeps); 0: none.
std::atomic<int> g_tuning[SDKDE_TUNE_COUNT];

int tuning(int knob, int fallback)
{
    const int v = g_tuning[knob].load(std::memory_order_relaxed);
    return v > 0 ? v : fallback;
}

// Workgroups needed to keep 256 CUs busy with a few waves per SIMD (tiny problems).
constexpr int64_t kTargetBlocks = 2048;
constexpr int kComputeUnits = 256;

// Relative cost per unit of work of running the matrix-path kernels with `ni` row tiles per wave instead of the
// best count (operand reuse against register pressure), measured on MI355X: the fp32 mode by the figures at half_shape, the
// fp16 input modes at n = 131072 resp. n = 262144, m = 65536.
double row_tiles_penalty(bool score, int kb, int ni, uint32_t prec)
{
    if (prec != SDKDE_PREC_FP32) {
        // The cheap MFMAs leave the operand loads and the VALU work exposed, so few row tiles cost much.  Score, fp16x2:
        // d = 16 2 / 4 / 8 row tiles 6.51 / 6.02 / 6.13 ms, d = 32 2 / 4: 12.1 / 10.7, d = 64: 24.0 / 21.7; fp16x2-all
        // (d = 16 only): 9.88 / 5.25 / 4.36 ms.  Eval: d = 16 2 / 4 / 8 / 16: 3.01 / 2.41 / 2.27 / 2.95 ms,
        // d = 32 2 / 4 / 8: 8.15 / 4.30 / 3.39, d = 64 2 / 4: 15.3 / 7.9 ms.
        if (score && (prec == SDKDE_PREC_FP16X2_ALL || prec == SDKDE_PREC_FP16X2_PHI16)) return ni >= 8 ? 1.0 : ni == 4 ? 1.2 : 2.25;
        if (score) return kb >= 5 ? 1.0 : kb == 1 ? (ni >= 8 ? 1.018 : ni == 4 ? 1.0 : 1.08) : (ni >= 4 ? 1.0 : 1.12);
        if (kb == 1) return ni == 16 ? 1.32 : ni == 8 ? 1.0 : ni == 4 ? 1.065 : 1.33;
        if (kb == 2) return ni == 8 ? 1.0 : ni == 4 ? 1.27 : 2.4;
        return kb >= 5 ? 1.0 : ni == 4 ? 1.0 : 1.94;
    }
    if (score) {
        if (kb == 1) return ni == 8 ? 1.0 : ni == 4 ? 1.01 : 1.05;
        return ni == 4 ? 1.0 : kb == 6 ? 1.3 : kb == 3 ? 1.06 : 1.04;
    }
    if (kb == 1) return ni == 8 ? 1.0 : ni == 4 ? 1.03 : 1.1;
    return ni == 4 || kb == 8 ? 1.0 : kb >= 6 ? 1.07 : 1.05;
}

// Estimated time of the pair kernel plus its share of the epilogue for `ni` row tiles per wave and `nsplit`
// splits, in units of one wave's time for one 16 x 16 tile.  A compute unit works through its
// ceil(workgroups / 256) workgroups at a rate that does not depend on how many are resident (the kernels are
// bound by instruction issue), so the time is rounds x (work of a workgroup), plus a tail that grows with the
// length of a workgroup, plus the traffic of one more partial slot per split (written once, read once, at about
// 3 TB/s).  Fitted to sweeps over (ni, nsplit) at d = 16 .. 128, n = 8192 .. 1048576, m = 1024 .. 200000: the
// pick is within 0.3 % of the best measured pair on average (2.3 % at worst), where "as many workgroups as
// fill the chip eight times" was 4.7 % off on average and up to 28 % at n = 8192 .. 24576.
double plan_cost(bool score, int kb, uint32_t prec, int64_t m, int64_t m_pad, int ntiles, int ni, int nsplit)
{
    const int64_t row_blocks = (m + kWavesPerBlock * kTile * ni - 1) / (kWavesPerBlock * kTile * ni);
    const int64_t groups = row_blocks * nsplit;
    const int64_t rounds = (groups + kComputeUnits - 1) / kComputeUnits;
    int tps = (ntiles + nsplit - 1) / nsplit;
    tps += tps & 1;
    const double slot_bytes = (double)m_pad * (score ? 16 * kb + 1 : 1) * 8.0;
    if (prec == SDKDE_PREC_FP32) {
        // pair_half_kernel, with the constants that sweeps at n = 600 .. 100000 gave for three-part operands (its tiles are a
        // third shorter; plans, and with them the sizes that workspaces are asked for, stay what they were): four (eval: one) tiles' time to start a workgroup; waves of
        // several workgroups are needed on a SIMD to overlap its matrix and vector work (score at n = 4096, d = 16: one
        // workgroup per compute unit 23.6 us, two 21.3; eval at 32768 x 4096: two 43.3 us, four 38.9); long workgroups
        // leave eval a longer tail (65536 x 8192: four per unit 118 us, eight 114); a slot moves at 6 TB/s.
        double work = (double)rounds * ni * (tps + (score ? 4.0 : 1.0)) * row_tiles_penalty(score, kb, ni, prec);
        const int64_t waves = rounds * half_shape(kb, score, ni).waves / 4;
        if (waves == 1) work *= 1.3;
        else if (score && kb == 1 && waves == 2) work *= 1.02;
        else if (!score && kb <= 2 && waves <= 3) work *= waves == 2 ? 1.1 : 1.04;
        const double tile_clk = score ? 115.0 + 130.0 * kb : 45.0 + 62.0 * kb;
        return work + (score ? 0.11 : 0.25) * ni * tps + nsplit * slot_bytes / 2500.0 / tile_clk;
    }
    const double work = (double)rounds * ni * (tps + 1.0) * row_tiles_penalty(score, kb, ni, prec);
    const double tail = 0.1 * ni * tps;
    // clocks per tile, in proportion to the measured kernel times, from those of an fp32 MFMA kernel
    double tile_clk = 33.0 * (score ? 8 : 4) * kb + 50.0;
    if (prec == SDKDE_PREC_FP16X2) tile_clk *= 0.62;
    if (prec == SDKDE_PREC_FP16X2_ALL) tile_clk *= score ? 0.41 : 0.62;
    if (prec == SDKDE_PREC_FP16X2_PHI16) tile_clk *= score ? 0.36 : 0.62;
    const double slot = slot_bytes / 1250.0 / tile_clk;          // 1250 bytes per clock = 3 TB/s at 2.4 GHz
    return work + tail + nsplit * slot;
}

// The same estimate for the thin path (rows per thread `r`, 256 r rows per workgroup), in units of one thread's
// time for one row against one 16-sample tile.  One row per thread is the fastest form per pair (measured at
// n = 262144: d = 1 score 9.96 / 10.36 / 10.23 ms with 1 / 2 / 4 rows, d = 3 18.2 / 18.7 / 19.8 ms), and the
// tail weighs more than on the matrix path; fitted to sweeps at d = 1 and 3, n = 8192 .. 1048576: the pick is
// within 0.2 % of the best measured pair on average (1.3 % at worst), the earlier rule was 7 % off on average.
double plan_cost_thin(bool score, int d, int64_t m, int64_t m_pad, int ntiles, int r, int nsplit)
{
    const int64_t row_blocks = (m + (int64_t)kBlock * r - 1) / ((int64_t)kBlock * r);
    const int64_t groups = row_blocks * nsplit;
    const int64_t rounds = (groups + kComputeUnits - 1) / kComputeUnits;
    int tps = (ntiles + nsplit - 1) / nsplit;
    tps += tps & 1;
    const double penalty = r == 1 ? 1.0 : r == 2 ? 1.0 + 0.015 * (1 + d) : 1.0 + 0.03 * d;
    const double work = (double)rounds * r * (tps + 1.0) * penalty;
    const double tail = 0.6 * r * tps;
    // clocks per row and tile: 16 pairs of 3d + 3 (score) or 2d + 3 (eval) VALU issue slots of 4 clocks
    const double tile_clk = 64.0 * (score ? 3 * d + 3 : 2 * d + 3);
    const double slot = (double)m_pad * (score ? d + 1 : 1) * 8.0 / 1250.0 / tile_clk;
    return work + tail + nsplit * slot;
}

int most_row_tiles(int kb, bool score, uint32_t prec)
{
    return prec == SDKDE_PREC_FP32 ? max_half_rt(kb, score) : max_row_tiles(kb, score ? kScoreSelf : kEval, (int)prec);
}

Plan make_plan(int64_t n, int64_t m, int d, bool score, uint32_t flags)
{
    Plan p{};
    p.d = d;
    // Direct differences on the VALU: up to d = 6 for the score kinds, up to d = 3 for eval, because they have no
    // Gram-expansion error.  It is not the faster form everywhere: at n = 262144, m = 65536, fp32, VALU / matrix form, score
    // d = 4 19.7 / 23.4 ms, d = 5 22.9 / 23.5, d = 6 26.9 / 23.6; eval d = 1 2.04 / 2.80, d = 2 2.59 / 2.64, d = 3
    // 3.22 / 2.63; at 4000 x 3000 the matrix form is ahead from d = 1 (eval 23.5 / 16.9 us, score d = 4 35.1 / 21.3).
    p.thin = d <= (score ? kThinMaxDScore : kThinMaxDEval);
    p.dp = p.thin ? d : (int)round_up(d, 16);
    p.n_pad = round_up(n, kRowPad);
    p.m_pad = round_up(m > 0 ? m : 1, kRowPad);
    p.ntiles = (int)((n + 2 * kTile - 1) / (2 * kTile)) * 2;   // even: the pair kernel alternates two operand sets
    // at least 16 tiles per split; the fp32 mode's kernels take 4 (score at n = 600, d = 8: 8 splits 14.2 us, 2 splits 17.8;
    // eval at 4096 x 512, d = 64: 64 splits 15.9 us, 16 splits 20.7)
    const uint32_t prec = effective_prec(flags, false, p.dp);
    p.parts = !p.thin && prec == SDKDE_PREC_FP32;
    const int least_tiles = p.parts ? 4 : 16;
    const int max_split = p.ntiles >= 2 * least_tiles ? p.ntiles / least_tiles : 1;

    // Candidate row-tile counts, largest (most operand reuse) first.
    int cand[5];
    int nc = 0;
    if (p.thin && d > kThinMaxDEval) {
        cand[nc++] = 1;                 // built with one row per thread only
    } else if (p.thin) {
        cand[nc++] = 4; cand[nc++] = 2; cand[nc++] = 1;
    } else {
        const int kb = p.dp / 16;
        for (int v = most_row_tiles(kb, score, effective_prec(flags, false, p.dp)); v >= 2; v /= 2) cand[nc++] = v;
    }
    const int forced_ni = tuning(score ? SDKDE_TUNE_SCORE_ROW_TILES : SDKDE_TUNE_EVAL_ROW_TILES, 0);
    int forced_split = tuning(score ? SDKDE_TUNE_SCORE_SPLITS : SDKDE_TUNE_EVAL_SPLITS, 0);
    if (forced_split > p.ntiles) forced_split = p.ntiles;
    {
        // a forced value must be one the dispatch tables below instantiate
        const int kb = p.thin ? 0 : p.dp / 16;
        const int widest = p.thin ? (d > kThinMaxDEval ? 1 : 4)
                                  : most_row_tiles(kb, score, effective_prec(flags, false, p.dp));
        const int narrowest = p.thin ? 1 : 2;
        if (forced_ni >= narrowest && forced_ni <= widest && (forced_ni & (forced_ni - 1)) == 0) {
            cand[0] = forced_ni;
            nc = 1;
        }
    }
    auto set_row_tiles = [&](int ni) {
        p.ni = ni;
        p.rows_per_block = p.thin ? kBlock * ni : kWavesPerBlock * kTile * ni;
        p.row_blocks = (m + p.rows_per_block - 1) / p.rows_per_block;
        if (p.row_blocks < 1) p.row_blocks = 1;
    };

    if (max_split >= 8 || p.parts) {
        // Enough samples for one group of splits per XCD: the (row tiles or rows per thread, splits) pair of least
        // estimated time; ties go to more rows per workgroup, then fewer splits.  Up to n = 16384 the fp32 mode's
        // kernels may take fewer splits too: whole rounds of workgroups then count for more than each XCD streaming an
        // eighth of the samples.  Score with 7 / 8 / 16 splits at n = 9000: d = 16 50 / 56 / 52 us, d = 64 116 / 148 / 126,
        // d = 128 254 / 325 / 281; with 4 / 8 / 16 at n = 16000: d = 64 310 / 297 / 311, d = 128 682 / 704 / 758.
        const int most = max_split >= 8 ? (max_split / 8 * 8 < 1024 ? max_split / 8 * 8 : 1024) : max_split;
        const int first = forced_split > 0 ? forced_split : p.parts && p.ntiles <= 1024 ? 1 : 8;
        const int last = forced_split > 0 ? forced_split : most;
        double best = 0.0;
        int best_ni = 0, best_split = 0;
        for (int k = 0; k < nc; ++k) {
            for (int sp = first; sp <= last; sp += sp < 8 ? 1 : 8) {
                const double c = p.thin ? plan_cost_thin(score, d, m > 0 ? m : 1, p.m_pad, p.ntiles, cand[k], sp)
                                        : plan_cost(score, p.dp / 16, prec, m > 0 ? m : 1, p.m_pad, p.ntiles, cand[k], sp);
                if (best_ni == 0 || c < best) {
                    best = c;
                    best_ni = cand[k];
                    best_split = sp;
                }
            }
        }
        set_row_tiles(best_ni);
        p.nsplit = best_split;
    } else {
        // Tiny sample sets: the largest row count per workgroup that still gives the chip enough workgroups,
        // with as many splits as that takes.
        for (int k = 0; k < nc; ++k) {
            set_row_tiles(cand[k]);
            int64_t want = (kTargetBlocks + p.row_blocks - 1) / p.row_blocks;
            if (max_split >= 8) {                       // one group of splits per XCD
                want = round_up(want < 8 ? 8 : want, 8);
                if (want > max_split) want = max_split / 8 * 8;
            } else if (want > max_split) {
                want = max_split;
            }
            p.nsplit = (int)want;
            if (forced_split > 0) p.nsplit = forced_split;
            if (p.row_blocks * p.nsplit >= kTargetBlocks / 2) break;
        }
    }
    p.tiles_per_split = (p.ntiles + p.nsplit - 1) / p.nsplit;
    p.tiles_per_split += p.tiles_per_split & 1;
    return p;
}

// Row tiles per wave of the pair_sym_kernel instantiation for kb 16-column blocks; 0: not built, the flag is ignored.
// (With dp >= 48 its operands leave no room for two waves per SIMD.)
constexpr int sym_row_tiles(int kb, int prec)
{
    return prec != SDKDE_PREC_FP32 ? 0 : kb == 1 ? 4 : kb == 2 ? 2 : 0;
}
// Least rows of a sample block, which are also what the smallest block size is a multiple of.
constexpr int sym_least_rows(int kb) { return kb == 1 ? 1024 : 512; }

// Most groups of sample blocks in the symmetric mode (a row gets one partial slot per group, plus three).
constexpr int kSymMaxGroups = 64;

// Decomposition of the symmetric mode, if this call takes it: the score at the samples themselves on the
// matrix path, for the dimensions and input modes pair_sym_kernel is built for (sym_row_tiles).  Block size:
// as many rows as the LDS accumulators hold ((dp + 1) floats per row within ~136 KiB), halved while there
// would be too few items to fill the chip.
void apply_symmetric(Plan& p, int64_t n, uint32_t flags, bool self)
{
    if (!(flags & SDKDE_FLAG_SYMMETRIC) || !self || p.thin) return;
    const int kb = p.dp / 16;
    const int ni = sym_row_tiles(kb, (int)(flags & 15u));
    if (ni == 0) return;
    p.sym_ni = ni;
    const int sb = sym_least_rows(kb);
    int rb = kb == 1 ? 2048 : kb == 2 ? 1024 : 512;
    auto items = [&](int rb_) {
        int64_t nb = (n + rb_ - 1) / rb_;
        if (nb > kSymMaxGroups) nb = kSymMaxGroups;
        return nb * (nb + 1) / 2;
    };
    while (rb > sb && items(rb) < 1024) rb /= 2;
    const int forced_rb = tuning(SDKDE_TUNE_SYM_BLOCK_ROWS, 0);
    if (forced_rb >= sb && forced_rb <= rb * 8 && forced_rb % sb == 0 && (forced_rb & (forced_rb - 1)) == 0 &&
        sym_lds_bytes(kb, forced_rb) <= 160 * 1024)
        rb = forced_rb;
    int max_groups = tuning(SDKDE_TUNE_SYM_GROUPS, kSymMaxGroups);
    if (max_groups < 1 || max_groups > kSymMaxGroups) max_groups = kSymMaxGroups;
    const int64_t n_pad = round_up(n, rb > kRowPad ? rb : kRowPad);
    const int64_t nblocks = n_pad / rb;
    if (nblocks > (1 << 20)) return;
    const int per_group = (int)((nblocks + max_groups - 1) / max_groups);
    const int ngroups = (int)((nblocks + per_group - 1) / per_group);
    // Below 512 work items (two rounds of one per CU) the ordinary kernels are well ahead and the flag is ignored
    // (SDKDE_TUNE_SYM_MIN_ITEMS: for tests of the mode at small sizes).  The line is where the mode began to pay with fp32
    // MFMAs, and callers that set the flag get the mode, its workspace and its summation order from there on; with
    // the ordinary kernels on two fp16 parts it no longer pays: its own are on three bf16 parts, and the vector work it
    // halves and the matrix work it cuts by a quarter have become cheaper than its transposes, folds and phase barriers.
    // Score, symmetric / ordinary: d = 16 n = 32768 482 / 387 us, 131072 5.99 / 4.76 ms, 262144 23.4 / 18.5; d = 8 n = 131072
    // 5.99 / 4.38 ms; d = 32 n = 16384 229 / 130 us, 100000 6.27 / 3.87 ms.
    int min_items = tuning(SDKDE_TUNE_SYM_MIN_ITEMS, 512);
    if (min_items < 1) min_items = 1;
    if ((int64_t)ngroups * (ngroups + 1) / 2 < min_items) return;
    p.sym_on = true;
    p.sym_rb = rb;
    p.sym_nblocks = (int)nblocks;
    p.sym_per_group = per_group;
    p.sym_ngroups = ngroups;
    p.n_pad = p.m_pad = n_pad;          // whole blocks; the points are the samples
}

struct Workspace {
    float* centre;                         // the point all coordinates are taken relative to (prep.h)
    uint64_t* stamp;                       // record of the last sample preparation (prep.h)
    float* xs;  float* xt;  float* xn;     // samples: scaled rows, blocked transpose, -|x|^2
    float* ps;  float* pn;                 // evaluation points (alias xs/xn when they are the samples)
    float* residual;                       // of points held in two parts, behind their rows (half2.h)
    float* shift;                          // per-point exponent shift of the max-shifted mode (separate points only)
    float* part_t;  float* part_d;
    float* part_shift;                     // a shift a slot and point (max-shifted sums of the two-part format; a single slot's: `shift`)
    size_t bytes;
};

// Lays out the workspace for `plan`; base may be null (size query).  separate_points: the
// evaluation points are an array of their own (eval, or score at points != samples).
Workspace layout(const Plan& p, bool score, bool separate_points, void* base, uint32_t flags = 0)
{
    Workspace w{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return base ? (char*)base + at : (char*)nullptr;
    };
    w.centre = (float*)take(sizeof(float) * SDKDE_MAX_D);
    w.stamp = (uint64_t*)take(sizeof(uint64_t) * kStampWords);
    const int format = operand_format(p, flags);
    auto rows_floats = [&](int64_t rows) { return (size_t)(p.parts ? split3_floats(rows, p.dp) : rows * p.dp); };
    w.xs = (float*)take(sizeof(float) * rows_floats(p.n_pad));
    // blocked transpose for the second contraction: as the rows, or hi/lo fp16 pairs stored twice (2x the bytes)
    const size_t xt_scale = format == SDKDE_PREC_FP16X2_ALL ? 2 : 1;
    w.xt = (score && !p.thin) ? (float*)take(sizeof(float) * xt_scale * rows_floats(p.n_pad)) : nullptr;
    w.xn = (float*)take(sizeof(float) * p.n_pad);
    if (separate_points) {
        w.ps = (float*)take(sizeof(float) * rows_floats(p.m_pad));
        if (format == kFormatHalf2) w.residual = half2_residual(w.ps, p.m_pad, p.dp);
        w.pn = (float*)take(sizeof(float) * p.m_pad);
        w.shift = (float*)take(sizeof(float) * p.m_pad);
    } else {
        w.ps = w.xs;
        w.pn = w.xn;
    }
    // one slot per split
    size_t slots = (size_t)p.nsplit;
    if (p.sym_on) slots = (size_t)p.sym_ngroups + 2;     // pair_sym_kernel's, then the in-block pass
    w.part_t = score ? (float*)take(sizeof(float) * slots * p.m_pad * p.dp) : nullptr;
    w.part_d = (float*)take(sizeof(float) * slots * p.m_pad);
    if (separate_points && format == kFormatHalf2 && (flags & SDKDE_FLAG_MAX_SHIFT))
        w.part_shift = slots > 1 ? (float*)take(sizeof(float) * slots * p.m_pad) : w.shift;
    w.bytes = off;
    return w;
}

// Most samples of a call whose rows are summed whole, and most of them times 16-column blocks (whole_row_tiles).
constexpr int64_t kWholeSamples = 3072, kWholeBlocks = 6144;

// Calls that would run on the FP16X2 kernels, whose Phi X is on the fp32 matrix units, are served by the fp32 mode's on two fp16
// parts, where the buffer holds their operands (6 bytes a value instead of 4) with the fewest splits, whatever the number of points,
// so that calls on one buffer agree on it; one of the size that sdkde_workspace_bytes gives holds them with all splits.  So are calls in the
// other fp16 modes on few samples, for which the fp32 mode has fewer launches.  FP16X2 / fp32 mode: one call, 20000 x 5003, d = 8
// 193 / 153 us, 16 192 / 170, 24 342 / 221, 64 673 / 377, 128 1364 / 851; eval d = 16 29.1 / 28.0, 64 90 / 48; 600 x 100, d = 16
// 26.4 / 18.0; score, n = 1048576, d = 16 376 / 289 ms.  Errors against 64-bit sums, 600 .. 30000 samples, d = 4 .. 128: at most 1.0
// of theirs, in the mean 0.72 on scores, 0.80 on log densities, 0.55 on Laplace-corrected ones.
// two_part_form: the flags such a call then runs with, the mode it would have run in kept in bits above the caller's (it is part of the
// record of prepared samples); those of other calls unchanged.  flags: of the kind of call (anchored_flags).
constexpr int kOwnModeShift = 16;
uint32_t two_part_form(uint32_t flags, int64_t n, int d, bool score)
{
    const int dp = (int)round_up(d, 16);
    if ((flags & 15u) == SDKDE_PREC_FP32 || d <= (score ? kThinMaxDScore : kThinMaxDEval) || (n > kWholeSamples && effective_prec(flags, false, dp) != SDKDE_PREC_FP16X2))
        return flags;
    return (flags & ~(15u | SDKDE_FLAG_SYMMETRIC)) | effective_prec(flags, false, dp) << kOwnModeShift;
}
uint32_t two_part_flags(uint32_t flags, int64_t n, int d, bool score, bool self, size_t workspace_bytes)
{
    const uint32_t as_fp32 = two_part_form(flags, n, d, score);
    if (as_fp32 == flags) return flags;
    Plan least{};
    least.parts = true;
    least.d = d;
    least.dp = (int)round_up(d, 16);
    least.n_pad = round_up(n, kRowPad);
    least.m_pad = self ? least.n_pad : kRowPad;
    least.nsplit = 1;
    return layout(least, score, !self, nullptr, as_fp32).bytes <= workspace_bytes ? as_fp32 : flags;
}

// Whether two of the caller's arrays share no byte (null: an array that is not there).
bool apart(const void* x, size_t nx, const void* y, size_t ny)
{
    return !x || !y || (const char*)x + nx <= (const char*)y || (const char*)y + ny <= (const char*)x;
}

bool bad_bandwidth(double h) { return !(h > 0.0) || !isfinite(h); }

// One group of splits per XCD, or a single split for tiny sample sets and on the matrix path: there a buffer may have been
// made for a plan with fewer splits (the fp32 mode takes five at 13000 samples of d = 16) and is used in another mode, and
// the fp32 mode's prepared rows are half as large again, so that calls may have to give up more slots for them.
inline int least_splits(const Plan& p) { return p.ntiles >= 128 && p.thin ? 8 : 1; }

// For a workspace smaller than the plan's own decomposition needs (a buffer sized for another m, say): halves the
// splits, down to least_splits.  False when already there.  Fewer
// splits mean fewer partial-sum slots; the call is then slower for few points but needs less memory.
bool fewer_splits(Plan& p)
{
    if (p.sym_on || p.nsplit <= least_splits(p)) return false;
    int s = p.nsplit / 2;
    if (s >= 8) s = s / 8 * 8;
    p.nsplit = s < least_splits(p) ? least_splits(p) : s;
    p.tiles_per_split = (p.ntiles + p.nsplit - 1) / p.nsplit;
    p.tiles_per_split += p.tiles_per_split & 1;
    return true;
}

// Lays the call's plan out in `bytes` bytes at base, with fewer splits if it has to; false: does not fit.
bool fit_workspace(Plan& p, bool score, bool separate_points, void* base, size_t bytes, uint32_t flags, Workspace* w)
{
    *w = layout(p, score, separate_points, base, flags);
    while (w->bytes > bytes && fewer_splits(p)) *w = layout(p, score, separate_points, base, flags);
    return w->bytes <= bytes;
}

// As above for separate points in the fp32 mode, which takes 6 bytes a value of a prepared point.  A buffer that
// would hold the call with 4 bytes a value (640000 queries at dp = 16, one split: 49 MB, with 6 bytes 69 MB) serves it all
// the same, the points in equal batches of whole workgroups' rows, one pass after the other; the plan is then one batch's.
// Smaller buffers are refused.  Returns the points of a batch (m: all of them); 0: does not fit.
int64_t fit_points(Plan& p, bool score, void* base, size_t bytes, uint32_t flags, int64_t m, Workspace* w)
{
    if (fit_workspace(p, score, true, base, bytes, flags, w)) return m;
    if (!p.parts) return 0;
    Plan four_bytes = p;
    four_bytes.parts = false;
    if (layout(four_bytes, score, true, base, flags).bytes > bytes) return 0;
    const int64_t all = p.row_blocks;
    auto fits = [&](int64_t blocks) {
        p.row_blocks = blocks;
        p.m_pad = blocks * p.rows_per_block;
        *w = layout(p, score, true, base, flags);
        return w->bytes <= bytes;
    };
    int64_t most = 0, over = all + 1;               // row blocks known to fit, and known (or taken) not to
    while (over - most > 1) {
        const int64_t mid = most + (over - most) / 2;
        (fits(mid) ? most : over) = mid;
    }
    if (most == 0) return 0;
    const int64_t batches = (all + most - 1) / most;
    fits((all + batches - 1) / batches);
    return p.m_pad;
}

// Bytes that hold the largest of: score at the samples themselves, score at m separate points, eval at m queries, each with its own
// decomposition on the kernels of its mode; two_part: in the fp16 modes also on those that serve the call in their place.
size_t calls_bytes(int64_t n, int64_t m, int d, uint32_t flags, bool two_part)
{
    size_t need = 0;
    auto cover = [&](uint32_t of_call, bool score, bool self) {
        Plan p = make_plan(n, self ? n : m, d, score, of_call);
        if (self) apply_symmetric(p, n, of_call, true);
        const size_t b = layout(p, score, !self, nullptr, of_call).bytes;
        need = b > need ? b : need;
    };
    auto of_kind = [&](bool score, bool self) {
        const uint32_t own = score ? anchored_flags(flags, self) : flags, instead = two_part_form(own, n, d, score);
        cover(own, score, self);
        if (two_part && instead != own) cover(instead, score, self);
    };
    of_kind(true, true);
    if (m > 0) {
        of_kind(true, false);
        of_kind(false, false);
    }
    return need;
}

// Optional instrumentation: event pairs around the main pair kernel of each call.
constexpr int kProfileSlots = 256;
struct Profile {
    bool enabled = false;
    hipEvent_t ev[2][kProfileSlots][2] = {};   // [score|eval][launch][begin|end], created lazily
    int count[2] = {0, 0};
} g_profile;

#define SDKDE_HIP(call)                                   \
    do {                                                  \
        if ((call) != hipSuccess) return SDKDE_EDEVICE;   \
    } while (0)

// Host-side shape check of every pair kernel: the grid's size, and that every row it touches exists in the padded arrays.
int check_grid(const Plan& p)
{
    if ((int64_t)p.row_blocks * p.nsplit > 0x7fffffffLL) return SDKDE_EUNSUPPORTED;
    if (p.row_blocks * p.rows_per_block > p.m_pad || (int64_t)p.ntiles * kTile > p.n_pad) return SDKDE_EINVAL;
    return SDKDE_OK;
}

inline int launched() { return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE; }

template <int KIND>
int launch_thin(const Plan& p, const Workspace& w, const float* shift, hipStream_t st)
{
    const dim3 grid((unsigned)(p.row_blocks * p.nsplit)), block(kBlock);
    const float laplace_c0 = 1.0f + 0.5f * (float)p.d;
#define SDKDE_LAUNCH_THIN(D_, R_)                                                                          \
    hipLaunchKernelGGL((pair_thin_kernel<D_, R_, KIND>), grid, block, 0, st, w.ps, w.xs, w.part_t, w.part_d, \
                       p.ntiles, p.tiles_per_split, p.nsplit, p.m_pad, laplace_c0, shift)
// d = 4 .. 6: the kinds a score call runs (one row per thread)
#define SDKDE_LAUNCH_THIN_SCORE(D_)                                                                        \
    do {                                                                                                   \
        if constexpr (KIND == kScoreSelf || KIND == kScorePoints || KIND == kRowMax) SDKDE_LAUNCH_THIN(D_, 1); \
        else return SDKDE_EUNSUPPORTED;                                                                    \
    } while (0)
    switch (p.d * 10 + p.ni) {
        case 14: SDKDE_LAUNCH_THIN(1, 4); break;
        case 12: SDKDE_LAUNCH_THIN(1, 2); break;
        case 11: SDKDE_LAUNCH_THIN(1, 1); break;
        case 24: SDKDE_LAUNCH_THIN(2, 4); break;
        case 22: SDKDE_LAUNCH_THIN(2, 2); break;
        case 21: SDKDE_LAUNCH_THIN(2, 1); break;
        case 34: SDKDE_LAUNCH_THIN(3, 4); break;
        case 32: SDKDE_LAUNCH_THIN(3, 2); break;
        case 31: SDKDE_LAUNCH_THIN(3, 1); break;
        case 41: SDKDE_LAUNCH_THIN_SCORE(4); break;
        case 51: SDKDE_LAUNCH_THIN_SCORE(5); break;
        case 61: SDKDE_LAUNCH_THIN_SCORE(6); break;
        default: return SDKDE_EUNSUPPORTED;
    }
#undef SDKDE_LAUNCH_THIN_SCORE
#undef SDKDE_LAUNCH_THIN
    return launched();
}

// The fp32 mode at d >= 4 (score kinds d >= 7).  FAR: the max-shifted sums, whose points may lie beyond the fp16 range.
template <int KIND, bool FAR, int KB, int TAIL, int RT>
int launch_half_shape(const Plan& p, const Workspace& w, hipStream_t st)
{
    constexpr bool score = KIND == kScoreSelf || KIND == kScorePoints;
    constexpr HalfShape sh = half_shape(KB, score, RT, KIND == kScoreSelf, FAR, TAIL);
    if constexpr (sh.ni == 0) {
        return SDKDE_EUNSUPPORTED;
    } else {
        static_assert(sh.ni * sh.waves == 4 * RT, "64 rt rows per workgroup");
        hipLaunchKernelGGL((pair_half_kernel<KB, TAIL, sh.ni, sh.waves, sh.nb, sh.ahead, sh.minw, KIND, FAR>),
                           dim3((unsigned)(p.row_blocks * p.nsplit)), dim3(sh.waves * kWave), 0, st, w.ps, w.pn, w.xs, w.xt,
                           w.xn, w.part_t, w.part_d, p.ntiles, p.tiles_per_split, p.nsplit, p.m_pad,
                           1.0f + 0.5f * (float)p.d, w.part_shift);
        return launched();
    }
}

template <int KIND, bool FAR, int KB, int TAIL>
int launch_half_tail(const Plan& p, const Workspace& w, hipStream_t st)
{
    switch (p.ni) {
        case 8: return launch_half_shape<KIND, FAR, KB, TAIL, 8>(p, w, st);
        case 4: return launch_half_shape<KIND, FAR, KB, TAIL, 4>(p, w, st);
        case 2: return launch_half_shape<KIND, FAR, KB, TAIL, 2>(p, w, st);
        default: return SDKDE_EUNSUPPORTED;
    }
}

template <int KIND, bool FAR>
int launch_half(const Plan& p, const Workspace& w, hipStream_t st)
{
    const int tail = half_tail(p.d, KIND == kScoreSelf);
    const bool eight = tail == kTailEight, spare = tail == kTailSpare;
    switch (p.dp / 16) {
        case 1: return eight ? launch_half_tail<KIND, FAR, 1, kTailEight>(p, w, st) : launch_half_tail<KIND, FAR, 1, kTailSixteen>(p, w, st);
        case 2: return spare ? launch_half_tail<KIND, FAR, 2, KIND == kScoreSelf ? kTailNone : kTailSpare>(p, w, st) : launch_half_tail<KIND, FAR, 2, kTailNone>(p, w, st);
        case 3: return eight ? launch_half_tail<KIND, FAR, 3, kTailEight>(p, w, st) : launch_half_tail<KIND, FAR, 3, kTailSixteen>(p, w, st);
        case 4: return spare ? launch_half_tail<KIND, FAR, 4, kTailSpare>(p, w, st) : launch_half_tail<KIND, FAR, 4, kTailNone>(p, w, st);
        case 5: return eight ? launch_half_tail<KIND, FAR, 5, kTailEight>(p, w, st) : launch_half_tail<KIND, FAR, 5, kTailSixteen>(p, w, st);
        case 6: return spare ? launch_half_tail<KIND, FAR, 6, kTailSpare>(p, w, st) : launch_half_tail<KIND, FAR, 6, kTailNone>(p, w, st);
        case 7: return eight ? launch_half_tail<KIND, FAR, 7, kTailEight>(p, w, st) : launch_half_tail<KIND, FAR, 7, kTailSixteen>(p, w, st);
        case 8: return spare ? launch_half_tail<KIND, FAR, 8, kTailSpare>(p, w, st) : launch_half_tail<KIND, FAR, 8, kTailNone>(p, w, st);
        default: return SDKDE_EUNSUPPORTED;
    }
}

// Small sample sets: row tiles a workgroup's waves share in pair_whole_kernel, 0: the call takes the kernels with split slots.
// rows: evaluation points.  The line lies where a workgroup's reads of all samples and the rounds of workgroups cost what the saved
// launch does.  Split slots / whole rows, us a call, one after the other: one-call pass with n / 4 queries, d = 8 n = 3072 26.7 / 21.9, d = 16
// n = 600 25.1 / 18.0, 2048 23.3 / 22.0, 2560 26.6 / 23.8, 3072 26.9 / 25.5, 4096 29.1 / 29.6, d = 24 n = 3072 32.1 / 29.7, d = 64 512 27.2 / 21.6,
// 1536 32.3 / 30.0, d = 128 256 34.3 / 25.3, 768 38.8 / 32.9; score at the samples 2048 15.1 / 14.0, 3072 18.2 / 15.8, d = 64 1536 20.2 / 19.7, d = 128
// 768 23.7 / 21.9; score at 16000 points, d = 16, n = 3072 32.1 / 29.6, 1200 21.8 / 19.2 with two row tiles a wave.
// Scores at few points have split slots to fill the chip with, where whole rows leave it to a few workgroups, each with all samples:
// d = 24, n = 1536 at 64 points 15.2 / 15.3, 4096 points 19.1 / 16.3; n = 3072 64 points 17.1 / 19.9, 1024 18.6 / 19.3, 4096 23.6 / 20.0; d = 64, n = 1024
// 64 points 16.3 / 17.1, 1024 18.2 / 17.3; n = 1536 17.3 / 20.2, 20.0 / 19.9; d = 80, n = 1024 18.0 / 18.9, 20.8 / 19.3; d = 96, n = 1024 19.5 / 21.8, 22.2 / 21.2.
// Densities: from about 800 samples on (d <= 8: 2300) the kernels take longer and the call, which the launches bound, does not: d = 16,
// 64 queries, n = 1024 15.5 / 13.1, alone 25.9 / 26.7, from a graph 9.2 / 10.0; 2048 15.4 / 12.7, 26.3 / 28.0, 9.6 / 11.4; 3072 15.6 / 13.3, 26.7 / 29.5,
// 10.0 / 12.9.  The line is that of the one-call pass, whose densities a call on its prepared samples repeats to the bit.
int whole_row_tiles(const Plan& p, int64_t n, int64_t rows, bool score, bool self, bool shifted)
{
    if (!p.parts || p.sym_on || shifted) return 0;
    if (tuning(score ? SDKDE_TUNE_SCORE_ROW_TILES : SDKDE_TUNE_EVAL_ROW_TILES, 0) || tuning(score ? SDKDE_TUNE_SCORE_SPLITS : SDKDE_TUNE_EVAL_SPLITS, 0)) return 0;
    const int kb = p.dp / 16;
    int64_t most = kWholeBlocks;
    if (score && !self) {
        if (rows < 1024) most = kb <= 4 ? 3072 : 5120;
        else if (rows < 2048 && kb <= 4) most = 5120;
    }
    if (n > kWholeSamples || n * kb > most) return 0;
    return rows <= kComputeUnits * kTile ? 1 : kb == 1 && rows <= 4 * kComputeUnits * kTile ? 2 : 0;
}

// Whether a score call of the thin path is thin_whole_kernel's.  Split slots / this, us a call: 600 samples, d = 1 15.8 / 8.6, 2000, d = 6
// 41.9 / 12.5; 4096 d = 1 14.1 / 9.9, d = 6 28.0 / 21.8; 3072 at 8192 points d = 2 27.6 / 14.0, d = 6 57.7 / 28.2; 4096 at 8192 points, where
// the split slots are 16 instead of 8, d = 2 16.7 / 16.6, 4 22.5 / 19.7, 5 24.0 / 23.6 and d = 6 28.8 / 32.7, left for its error, 0.70 of theirs.
// The time grows with the pairs, at sixteen threads a row with reads of their own.
bool thin_whole(const Plan& p, int64_t n, int64_t rows, bool shifted)
{
    if (!p.thin || shifted || tuning(SDKDE_TUNE_SCORE_ROW_TILES, 0) || tuning(SDKDE_TUNE_SCORE_SPLITS, 0)) return false;
    return n <= 4096 && rows <= 8192;
}

int launch_thin_whole(const float* samples, int64_t n, const float* points, int64_t m, int d, double h, double a, float* score_out,
                      float* samples_sd_out, const Stamp& stamp, hipStream_t st)
{
    const dim3 grid((unsigned)((m + kThinWholeRows - 1) / kThinWholeRows)), block(kBlock);
#define SDKDE_LAUNCH_THIN_WHOLE(D_)                                                                                              \
    hipLaunchKernelGGL(thin_whole_kernel<D_>, grid, block, 0, st, samples, (int)n, points, m, (float)a, (float)(1.0 / (a * h * h)), \
                       least_trusted_sum(n), score_out, (float)(0.5 * h * h), samples_sd_out, stamp)
    switch (d) {
        case 1: SDKDE_LAUNCH_THIN_WHOLE(1); break;
        case 2: SDKDE_LAUNCH_THIN_WHOLE(2); break;
        case 3: SDKDE_LAUNCH_THIN_WHOLE(3); break;
        case 4: SDKDE_LAUNCH_THIN_WHOLE(4); break;
        case 5: SDKDE_LAUNCH_THIN_WHOLE(5); break;
        case 6: SDKDE_LAUNCH_THIN_WHOLE(6); break;
        default: return SDKDE_EUNSUPPORTED;
    }
#undef SDKDE_LAUNCH_THIN_WHOLE
    return launched();
}

// Lays a call of such a kernel out: as layout() does, without partial slots.
Workspace whole_layout(Plan p, bool score, bool separate_points, void* base, uint32_t flags)
{
    p.nsplit = 0;
    return layout(p, score, separate_points, base, flags);
}

template <int KIND, bool FIT, int KB, int TAIL>
int launch_whole_tail(const Plan& p, const Workspace& w, int row_tiles, int64_t m, const WholeOut& out, hipStream_t st)
{
    const int64_t rows = FIT ? p.n_pad : m, blocks = (rows + row_tiles * kTile - 1) / (row_tiles * kTile);
    // Host-side shape check: every row and chunk exists in the padded arrays, and no wave has more chunks than one level sums.
    if (blocks > 0x7fffffffLL || blocks * row_tiles * kTile > p.m_pad || (int64_t)p.ntiles * kTile > p.n_pad || p.ntiles % 2 ||
        p.ntiles / 2 > whole_waves(KB, row_tiles) * kWholeChunks)
        return SDKDE_EINVAL;
    const dim3 grid((unsigned)blocks), block(whole_waves(KB, row_tiles) * kWave);
#define SDKDE_LAUNCH_WHOLE(NI_)                                                                                              \
    hipLaunchKernelGGL((pair_whole_kernel<KB, TAIL, NI_, KIND, FIT>), grid, block, 0, st, w.ps, w.pn, w.xs, w.xt, w.xn,       \
                       p.ntiles / 2, p.n_pad, m, p.m_pad, 1.0f + 0.5f * (float)p.d, out)
    if (row_tiles == 1) {
        SDKDE_LAUNCH_WHOLE(1);
    } else if constexpr (KB == 1 && KIND != kScoreSelf) {           // (two: from more rows on than there are samples here)
        if (row_tiles != 2) return SDKDE_EUNSUPPORTED;
        SDKDE_LAUNCH_WHOLE(2);
    } else {
        return SDKDE_EUNSUPPORTED;
    }
#undef SDKDE_LAUNCH_WHOLE
    return launched();
}

template <int KIND, bool FIT = false>
int launch_whole(const Plan& p, const Workspace& w, int row_tiles, int64_t m, const WholeOut& out, hipStream_t st)
{
    const int tail = half_tail(p.d, KIND == kScoreSelf);
    const bool eight = tail == kTailEight, spare = tail == kTailSpare;
#define SDKDE_WHOLE_ODD(KB_) (eight ? launch_whole_tail<KIND, FIT, KB_, kTailEight>(p, w, row_tiles, m, out, st) : launch_whole_tail<KIND, FIT, KB_, kTailSixteen>(p, w, row_tiles, m, out, st))
#define SDKDE_WHOLE_EVEN(KB_) (spare ? launch_whole_tail<KIND, FIT, KB_, kTailSpare>(p, w, row_tiles, m, out, st) : launch_whole_tail<KIND, FIT, KB_, kTailNone>(p, w, row_tiles, m, out, st))
    switch (p.dp / 16) {
        case 1: return SDKDE_WHOLE_ODD(1);
        case 2: return spare ? launch_whole_tail<KIND, FIT, 2, KIND == kScoreSelf ? kTailNone : kTailSpare>(p, w, row_tiles, m, out, st) : launch_whole_tail<KIND, FIT, 2, kTailNone>(p, w, row_tiles, m, out, st);
        case 3: return SDKDE_WHOLE_ODD(3);
        case 4: return SDKDE_WHOLE_EVEN(4);
        case 5: return SDKDE_WHOLE_ODD(5);
        case 6: return SDKDE_WHOLE_EVEN(6);
        case 7: return SDKDE_WHOLE_ODD(7);
        case 8: return SDKDE_WHOLE_EVEN(8);
        default: return SDKDE_EUNSUPPORTED;
    }
#undef SDKDE_WHOLE_EVEN
#undef SDKDE_WHOLE_ODD
}

// The fp16 input modes.
template <int KIND, int PREC>
int launch_mfma(const Plan& p, const Workspace& w, const float* shift, hipStream_t st)
{
    const dim3 grid((unsigned)(p.row_blocks * p.nsplit)), block(kBlock);
    const float laplace_c0 = 1.0f + 0.5f * (float)p.d;
#define SDKDE_CASE_NI(KB_, NI_)                                                                                      \
    case NI_:                                                                                                        \
        if constexpr (NI_ <= max_row_tiles(KB_, KIND, PREC))                                                         \
            hipLaunchKernelGGL((pair_mfma_kernel<KB_, NI_, KIND, PREC>), grid, block, 0, st, w.ps, w.pn, w.xs, w.xt, \
                               w.xn, w.part_t, w.part_d, p.ntiles, p.tiles_per_split, p.nsplit, p.m_pad, laplace_c0, \
                               shift);                                                                               \
        else return SDKDE_EUNSUPPORTED;                                                                              \
        break;
    switch (p.dp / 16) {
        case 1:
            switch (p.ni) { SDKDE_CASE_NI(1, 16) SDKDE_CASE_NI(1, 8) SDKDE_CASE_NI(1, 4) SDKDE_CASE_NI(1, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 2:
            switch (p.ni) { SDKDE_CASE_NI(2, 8) SDKDE_CASE_NI(2, 4) SDKDE_CASE_NI(2, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 3:
            switch (p.ni) { SDKDE_CASE_NI(3, 4) SDKDE_CASE_NI(3, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 4:
            switch (p.ni) { SDKDE_CASE_NI(4, 4) SDKDE_CASE_NI(4, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 5:
            switch (p.ni) { SDKDE_CASE_NI(5, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 6:
            switch (p.ni) { SDKDE_CASE_NI(6, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 7:
            switch (p.ni) { SDKDE_CASE_NI(7, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        case 8:
            switch (p.ni) { SDKDE_CASE_NI(8, 2) default: return SDKDE_EUNSUPPORTED; }
            break;
        default: return SDKDE_EUNSUPPORTED;
    }
#undef SDKDE_CASE_NI
    return launched();
}

template <int KIND>
int launch_pair_prec(const Plan& p, const Workspace& w, uint32_t flags, const float* shift, hipStream_t st)
{
    const int rc = check_grid(p);
    if (rc != SDKDE_OK) return rc;
    // the thin-d path has no matrix inputs: it runs the same fp32 VALU code for every mode
    if (p.thin) return launch_thin<KIND>(p, w, shift, st);
    const uint32_t prec = effective_prec(flags, p.thin, p.dp);
    if (prec == SDKDE_PREC_FP32) {
        if constexpr (KIND == kScoreSelf) return launch_half<KIND, false>(p, w, st);
        else if constexpr (KIND == kRowMax) return SDKDE_EUNSUPPORTED;      // (these kernels find the shifts as they go)
        else return shift ? launch_half<KIND, true>(p, w, st) : launch_half<KIND, false>(p, w, st);
    }
    if constexpr (KIND == kScoreSelf || KIND == kScorePoints) {
        if (prec == SDKDE_PREC_FP16X2_ALL) return launch_mfma<KIND, SDKDE_PREC_FP16X2_ALL>(p, w, shift, st);
        if (prec == SDKDE_PREC_FP16X2_PHI16) return launch_mfma<KIND, SDKDE_PREC_FP16X2_PHI16>(p, w, shift, st);
    }
    // kinds without a second contraction: the fp16 modes are the same kernel
    return launch_mfma<KIND, SDKDE_PREC_FP16X2>(p, w, shift, st);
}

// Symmetric mode: pairs across blocks (pair_sym_kernel), then the pairs inside each block with the ordinary
// kernel restricted to the block (slot ngroups + 1).
template <int KB>
int launch_sym_kernel(const Plan& p, const Workspace& w, hipStream_t st)
{
    constexpr int NI = sym_row_tiles(KB, SDKDE_PREC_FP32);
    const size_t lds = sym_lds_bytes(KB, p.sym_rb);
    // Host-side shape check: whole blocks of whole workgroup row sets, a power of two of chunks per phase.
    if (p.sym_rb % (kSymWaves * NI * kTile) || p.sym_rb % (kSymWaves * kChunkRows) || (p.sym_rb & (p.sym_rb - 1)) ||
        (int64_t)p.sym_nblocks * p.sym_rb != p.n_pad || lds > 160 * 1024)
        return SDKDE_EINVAL;
    // more than 64 KiB of dynamic LDS has to be enabled per kernel and device; remembered, so that later calls
    // (also ones under stream capture) only launch
    constexpr int kMaxDevices = 64;
    static std::mutex guard;                          // host threads may call concurrently
    static size_t lds_allowed[kMaxDevices] = {};
    int dev = 0;
    SDKDE_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> lock(guard);
        if (dev < 0 || dev >= kMaxDevices || lds > lds_allowed[dev]) {
            SDKDE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&pair_sym_kernel<KB, NI>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            if (dev >= 0 && dev < kMaxDevices) lds_allowed[dev] = lds;
        }
    }
    const int64_t items = (int64_t)p.sym_ngroups * (p.sym_ngroups + 1) / 2;
    hipLaunchKernelGGL((pair_sym_kernel<KB, NI>), dim3((unsigned)items), dim3(kSymBlock), lds, st, w.xs, w.xt,
                       w.xn, w.part_t, w.part_d, p.n_pad, p.sym_rb, p.sym_nblocks, p.sym_per_group, p.sym_ngroups);
    int rc = launched();
    if (rc != SDKDE_OK) return rc;

    Plan band = p;
    band.nsplit = 1;
    band.tiles_per_split = p.sym_rb / kTile;        // the length of a block in tiles
    band.ni = 4;
    band.rows_per_block = kWavesPerBlock * kTile * band.ni;
    band.row_blocks = ((int64_t)p.ntiles * kTile + band.rows_per_block - 1) / band.rows_per_block;
    if (p.sym_rb % band.rows_per_block || (rc = check_grid(band)) != SDKDE_OK) return SDKDE_EINVAL;
    Workspace wb = w;                               // its slots follow pair_sym_kernel's
    wb.part_t = w.part_t + (size_t)(p.sym_ngroups + 1) * p.m_pad * p.dp;
    wb.part_d = w.part_d + (size_t)(p.sym_ngroups + 1) * p.m_pad;
    hipLaunchKernelGGL((pair_split_kernel<KB, 4, kWavesPerBlock, 4, true, 2>), dim3((unsigned)band.row_blocks), dim3(kBlock), 0, st,
                       wb.xs, wb.xt, wb.xn, wb.part_t, wb.part_d, band.ntiles, band.tiles_per_split);
    return launched();
}

int launch_symmetric(const Plan& p, const Workspace& w, hipStream_t st)
{
    switch (p.dp / 16) {
        case 1: return launch_sym_kernel<1>(p, w, st);
        case 2: return launch_sym_kernel<2>(p, w, st);
        default: return SDKDE_EUNSUPPORTED;
    }
}

// Launches an epilogue kernel (template parameter: threads per output) over `outputs` outputs of `nslots` slots.
#define SDKDE_LAUNCH_EPILOGUE_AS(nslots, outputs, st, MANY, FEW, ...)                                             \
    do {                                                                                                           \
        if (epilogue_parts(nslots, outputs) == kEpiPartsMany) {                                                    \
            constexpr int per_wg = kBlock / kEpiPartsMany;                                                         \
            hipLaunchKernelGGL((MANY), dim3((unsigned)(((outputs) + per_wg - 1) / per_wg)),                        \
                               dim3(kBlock), 0, st, __VA_ARGS__);                                                  \
        } else {                                                                                                   \
            constexpr int per_wg = kBlock / kEpiPartsFew;                                                          \
            hipLaunchKernelGGL((FEW), dim3((unsigned)(((outputs) + per_wg - 1) / per_wg)),                         \
                               dim3(kBlock), 0, st, __VA_ARGS__);                                                  \
        }                                                                                                          \
    } while (0)
#define SDKDE_COMMA ,
#define SDKDE_LAUNCH_EPILOGUE(KERNEL, nslots, outputs, st, ...) \
    SDKDE_LAUNCH_EPILOGUE_AS(nslots, outputs, st, KERNEL<kEpiPartsMany>, KERNEL<kEpiPartsFew>, __VA_ARGS__)
// As above for a kernel with a second parameter: whether slots have shifts of their own.
#define SDKDE_LAUNCH_SHIFTED_EPILOGUE(KERNEL, shifted, nslots, outputs, st, ...)                                                              \
    do {                                                                                                                                      \
        if (shifted) SDKDE_LAUNCH_EPILOGUE_AS(nslots, outputs, st, KERNEL<kEpiPartsMany SDKDE_COMMA true>, KERNEL<kEpiPartsFew SDKDE_COMMA true>, __VA_ARGS__);   \
        else SDKDE_LAUNCH_EPILOGUE_AS(nslots, outputs, st, KERNEL<kEpiPartsMany SDKDE_COMMA false>, KERNEL<kEpiPartsFew SDKDE_COMMA false>, __VA_ARGS__);         \
    } while (0)

// First pass of the max-shifted mode for separate points: row maxima of the exponent, then shift_kernel.  (The fp32 mode's matrix
// path has none.)
int launch_max_shift(const Plan& p, const Workspace& w, uint32_t flags, hipStream_t st)
{
    if (p.parts) return SDKDE_OK;
    int rc = launch_pair_prec<kRowMax>(p, w, flags, nullptr, st);
    if (rc != SDKDE_OK) return rc;
    SDKDE_LAUNCH_EPILOGUE(shift_kernel, p.nsplit, p.m_pad, st, w.part_d, p.nsplit, p.m_pad, w.shift,
                          p.thin ? nullptr : w.pn);
    return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE;
}

// Centre/scale/pad one or two arrays in a single launch (second.src == nullptr: only the first).
// centre_src: the samples whose strided subsample gives the centre (also left in w.centre); null: w.centre as an
// earlier launch on this workspace left it.
// What identifies prepared samples: the kind of call that prepared them (the score and eval layouts differ), the
// caller's array, its shape, the operand format and the coordinate scale as it reached the kernels.
Stamp make_stamp(const Workspace& w, bool check, bool score, const float* samples, int64_t n, int d, int format, float a, uint32_t flags)
{
    Stamp s{};
    s.where = w.stamp;
    s.check = check ? 1 : 0;
    uint32_t abits;
    memcpy(&abits, &a, sizeof abits);
    const uint64_t v[kStampWords] = {(score ? 1u : 2u) | flags >> kOwnModeShift << 8, (uint64_t)(uintptr_t)samples, (uint64_t)n, (uint64_t)d, (uint64_t)format, abits};
    for (int k = 0; k < kStampWords; ++k) s.value[k] = v[k];
    return s;
}

int launch_prep(const Plan& p, const PrepJob& first, const PrepJob& second, const float* centre_src, int64_t centre_n,
                double a, const Workspace& w, uint32_t flags, const Stamp& stamp, hipStream_t st)
{
    float* const units = operand_format(p, flags) == kFormatHalf2 && first.dst_t ? half2_units(first.dst, first.rows_pad, p.dp) : nullptr;
    const PrepCommon common = centre_of(centre_src, centre_n, p.d, w.centre, units);
    const int64_t per_block = p.thin ? kBlock : kPrepRows;
    if (first.rows_pad % per_block || (second.src && second.rows_pad % per_block)) return SDKDE_EINVAL;
    const int64_t blocks0 = first.rows_pad / per_block;
    const int64_t blocks1 = second.src ? second.rows_pad / per_block : 0;
    if (blocks0 + blocks1 > 0x7fffffffLL) return SDKDE_EUNSUPPORTED;
    const dim3 grid((unsigned)(blocks0 + blocks1)), block(kBlock);
    if (p.thin)
        hipLaunchKernelGGL(prep_thin_kernel, grid, block, 0, st, first, second, (int)blocks0, p.d, common, (float)a, stamp);
    else
    {
        const int format = operand_format(p, flags);
        const auto kernel = format != kFormatHalf2 ? prep_mfma_kernel<false, SDKDE_MAX_D> : p.dp <= 32 ? prep_mfma_kernel<true, 32> : prep_mfma_kernel<true, SDKDE_MAX_D>;
        hipLaunchKernelGGL(kernel, grid, block, prep_lds_bytes(p.dp, format), st, first, second, (int)blocks0, p.d, p.dp, common, a, format, stamp);
    }
    return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE;
}

int check_common(const void* samples, int64_t n, int64_t m, int32_t d, double h, uint32_t flags)
{
    if (!samples || n < 1 || m < 0 || d < 1 || bad_bandwidth(h)) return SDKDE_EINVAL;
    constexpr uint32_t known = 15u | SDKDE_FLAG_MAX_SHIFT | SDKDE_FLAG_SYMMETRIC | SDKDE_FLAG_SAMPLES_PREPARED;
    if (d > SDKDE_MAX_D || (flags & ~known) != 0 || (flags & 15u) > SDKDE_PREC_FP16X2_PHI16) return SDKDE_EUNSUPPORTED;
    if (n > (int64_t)1 << 34 || m > (int64_t)1 << 34) return SDKDE_EUNSUPPORTED;
    return SDKDE_OK;
}

// edge 0: before the main kernel of a call of kind `which`; edge 1: after it.
int profile_mark(int which, int edge, hipStream_t st)
{
    if (!g_profile.enabled || g_profile.count[which] >= kProfileSlots) return SDKDE_OK;
    hipEvent_t& e = g_profile.ev[which][g_profile.count[which]][edge];
    if (!e) SDKDE_HIP(hipEventCreate(&e));
    SDKDE_HIP(hipEventRecord(e, st));
    if (edge == 1) ++g_profile.count[which];
    return SDKDE_OK;
}

// What the score epilogue of sdkde_fit_eval needs in order to prepare the eval pass's operands in the same launch
// (score_epilogue_prep_kernel): where that pass expects its prepared samples and queries, and the record it leaves.
struct FusedPrep {
    PrepJob sd_job, q_job;
    Stamp stamp;
    bool whole_score;       // the score pass is pair_whole_kernel's
    bool whole;             // both passes are (plan_whole_fit), these their plans and places
    Plan score_plan, eval_plan;
    Workspace score_at, eval_at;
};

// Whether the one-call pass can fold the eval pass's preparation into the score epilogue, and with what.  Both passes
// must be on the matrix path with their own full decomposition fitting the workspace, the epilogue must be the
// four-part one, and everything the fused launch writes for the eval pass must lie where the score pass no longer
// reads: the prepared shifted samples over the prepared samples (a workgroup reads its rows before it overwrites
// them), their norms and the prepared queries inside the blocked transpose, which only the pair kernel reads.
// sflags, eflags: the two passes' own (anchored_flags, two_part_flags).
bool plan_fused_prep(const float* samples_sd, int64_t n, const float* queries, int64_t m, int32_t d, double h, void* workspace,
                     size_t workspace_bytes, uint32_t sflags, uint32_t eflags, FusedPrep* out)
{
    if (m <= 0 || (eflags & (SDKDE_FLAG_MAX_SHIFT | SDKDE_FLAG_SAMPLES_PREPARED)) || (sflags & SDKDE_FLAG_SYMMETRIC)) return false;
    if (tuning(SDKDE_TUNE_SEPARATE_PREP, 0) == 1) return false;
    Plan ps = make_plan(n, n, d, true, sflags);
    apply_symmetric(ps, n, sflags, true);
    const Plan pe = make_plan(n, m, d, false, eflags);
    if (ps.thin || pe.thin || ps.sym_on || ps.n_pad != pe.n_pad || ps.dp != pe.dp) return false;
    // One workgroup of the folded launch reduces 32 rows x dp/4 items in dp/8 passes, where the plain epilogue spreads
    // them over dp/8 workgroups: measured per pass of the whole call (folded / separate, same box), d = 16: n = 2048
    // 28.4 / 29.9 us, 4096 33.7 / 35.7, 8192 66.2 / 67.5, 32768 x 4096 662.3 / 665.0; d = 32: 4096 50.0 / 49.1;
    // d = 64: 4096 81.8 / 77.0; d = 128: 145.0 / 131.2.  It pays at dp = 16 only.
    if (ps.dp != 16) return false;              // (what the folded launch is built for, too)
    const int format = operand_format(pe, eflags);
    if (operand_format(ps, sflags) != format) return false;
    const Workspace ws = layout(ps, true, false, workspace, sflags);
    const Workspace we = layout(pe, false, true, workspace, eflags);
    if (ws.bytes > workspace_bytes || we.bytes > workspace_bytes) return false;
    if (epilogue_parts(ps.nsplit, n * (int64_t)d) != kEpiPartsFew) return false;
    if (ps.n_pad % kPrepRows || pe.m_pad % kPrepRows || (ps.n_pad + pe.m_pad) / kPrepRows > 0x7fffffffLL) return false;
    const char* dead_begin = (const char*)ws.xt;
    const char* dead_end = (const char*)ws.xn;                   // the blocked transpose ends where the norms begin
    const char* wr_begin = (const char*)we.xn;
    const char* wr_end = (const char*)(we.pn + pe.m_pad);
    if (we.xs != ws.xs || wr_begin < dead_begin || wr_end > dead_end) return false;
    if ((const char*)we.ps < (const char*)(we.xn + pe.n_pad)) return false;
    const double a = operand_scale(format, h);
    out->sd_job = PrepJob{samples_sd, n, pe.n_pad, we.xs, nullptr, we.xn, kPadCoord, true, false, half_tail(d, false)};
    out->q_job = PrepJob{queries, m, pe.m_pad, we.ps, nullptr, we.pn, 0.0f, false, false, half_tail(d, false)};
    out->stamp = make_stamp(we, false, false, samples_sd, n, d, format, (float)a, eflags);
    return true;
}

// Whether the one-call pass is that of small sample sets whose two passes are pair_whole_kernel's (whole_row_tiles): three launches, the queries prepared with
// the samples, the shifted samples by the workgroups that form them.  The eval pass's operands stand where a call of its own has
// them (a later one may rely on the record, SDKDE_FLAG_SAMPLES_PREPARED), the score pass's behind them.
bool plan_whole_fit(const float* samples_sd, int64_t n, const float* queries, int64_t m, int32_t d, double h, void* workspace,
                    size_t workspace_bytes, uint32_t sflags, uint32_t eflags, FusedPrep* out)
{
    if (m <= 0 || (eflags & (SDKDE_FLAG_MAX_SHIFT | SDKDE_FLAG_SAMPLES_PREPARED)) || tuning(SDKDE_TUNE_SEPARATE_PREP, 0) == 1) return false;
    Plan& ps = out->score_plan = make_plan(n, n, d, true, sflags);
    apply_symmetric(ps, n, sflags, true);
    out->whole_score = whole_row_tiles(ps, n, n, true, true, false) != 0;
    if (!out->whole_score) return false;
    Plan& pe = out->eval_plan = make_plan(n, m, d, false, eflags);
    if (!whole_row_tiles(pe, n, m, false, false, false) || ps.n_pad != pe.n_pad) return false;
    // accepted or refused as the passes one by one are
    Workspace unused;
    Plan score_plan = ps, eval_plan = pe;
    if (!fit_workspace(score_plan, true, false, workspace, workspace_bytes, sflags, &unused) ||
        fit_points(eval_plan, false, workspace, workspace_bytes, eflags, m, &unused) != m)
        return false;
    const Workspace& we = out->eval_at = whole_layout(pe, false, true, workspace, eflags);
    Workspace& ws = out->score_at = whole_layout(ps, true, false, (char*)workspace + we.bytes, sflags);
    if (we.bytes + ws.bytes > workspace_bytes) return false;
    ws.centre = we.centre;
    ws.stamp = we.stamp;
    out->whole = true;
    const int format = operand_format(pe, eflags);
    out->sd_job = PrepJob{samples_sd, n, pe.n_pad, we.xs, nullptr, we.xn, kPadCoord, true, false, half_tail(d, false)};
    out->q_job = PrepJob{queries, m, pe.m_pad, we.ps, nullptr, we.pn, 0.0f, false, false, half_tail(d, false)};
    out->stamp = make_stamp(we, false, false, samples_sd, n, d, format, (float)operand_scale(format, h), eflags);
    return true;
}

// What the one-call pass folds together, if anything.  (Plans cost 0.4 us each at n = 4096, 3 us at 2^20, in front of the first launch: the
// number of samples alone rules the small form out.)
bool plan_fit(const float* samples_sd, int64_t n, const float* queries, int64_t m, int32_t d, double h, void* workspace, size_t workspace_bytes,
              uint32_t flags, FusedPrep* out)
{
    const uint32_t sflags = two_part_flags(anchored_flags(flags, true), n, d, true, true, workspace_bytes);
    const uint32_t eflags = two_part_flags(flags, n, d, false, false, workspace_bytes);
    if (n <= kWholeSamples) {
        if (plan_whole_fit(samples_sd, n, queries, m, d, h, workspace, workspace_bytes, sflags, eflags, out)) return true;
        if (out->whole_score) return false;         // (its kernel has its epilogue in it)
    }
    return plan_fused_prep(samples_sd, n, queries, m, d, h, workspace, workspace_bytes, sflags, eflags, out);
}

// One pass of a score call over the samples at m points (null: at the samples themselves, m = n).  samples_ready: they
// stand prepared in the workspace, by an earlier pass of the same call.
int score_pass(const Plan& p, const Workspace& w, const float* samples, int64_t n, const float* points, int64_t m, bool samples_ready,
               double h, float* score_out, float* samples_sd_out, uint32_t flags, hipStream_t st, const FusedPrep* fused, int whole_rows)
{
    int rc;
    const int d = p.d;
    const bool self = points == nullptr;
    const int format = operand_format(p, flags);
    const double a = operand_scale(format, h);
    // at the samples themselves the largest weight is the self pair (exponent 0): nothing to shift
    const bool shifted = !self && (flags & SDKDE_FLAG_MAX_SHIFT) != 0;
    // When the points are the samples (m == n, so m_pad == n_pad), one prepared array serves
    // as both operands.
    const PrepJob sample_job{samples, n, p.n_pad, w.xs, w.xt, w.xn, kPadCoord, true, shifted, half_tail(d, self)};
    // (a one-call pass of small sample sets prepares the eval pass's queries here)
    const PrepJob point_job = fused && whole_rows ? fused->q_job
                                                  : PrepJob{points, m, p.m_pad, w.ps, nullptr, w.pn, 0.0f, false, shifted, half_tail(d, false)};
    const Stamp stamp = make_stamp(w, samples_ready, true, samples, n, d, format, (float)a, flags);
    rc = samples_ready ? launch_prep(p, point_job, PrepJob{}, nullptr, 0, a, w, flags, stamp, st)
                       : launch_prep(p, sample_job, point_job, samples, n, a, w, flags, stamp, st);
    if (rc != SDKDE_OK) return rc;

    const float inv_ah2 = (float)(1.0 / (a * h * h)), half_h2 = (float)(0.5 * h * h);
    const ScoreUnits units{format == kFormatHalf2 ? half2_units(w.xs, p.n_pad, p.dp) : nullptr, self ? samples : points};
    const uintptr_t io = (uintptr_t)score_out | (uintptr_t)samples_sd_out | (samples_sd_out ? (uintptr_t)samples : 0);
    const int quad_io = (d % 4 == 0 && (io & 15) == 0) ? 1 : 0;
    if ((rc = profile_mark(0, 0, st)) != SDKDE_OK) return rc;
    if (whole_rows) {
        WholeOut out{};
        out.d = d;
        out.min_sum = least_trusted_sum(n);
        out.inv_ah2 = inv_ah2;
        out.half_h2 = half_h2;
        out.score = score_out;
        out.x = samples;
        out.x_sd = samples_sd_out;
        out.quad_io = quad_io;
        out.units = units;
        if (fused) {
            if (!self || !samples_sd_out) return SDKDE_EINVAL;
            out.sd_job = fused->sd_job;
            out.centre = w.centre;
            out.a = a;
            out.stamp = fused->stamp;
        }
        rc = fused  ? launch_whole<kScoreSelf, true>(p, w, whole_rows, m, out, st)
             : self ? launch_whole<kScoreSelf>(p, w, whole_rows, m, out, st)
                    : launch_whole<kScorePoints>(p, w, whole_rows, m, out, st);
        return rc != SDKDE_OK ? rc : profile_mark(0, 1, st);
    }
    if (shifted && (rc = launch_max_shift(p, w, flags, st)) != SDKDE_OK) return rc;
    const float* shift = shifted ? w.shift : nullptr;
    rc = p.sym_on ? launch_symmetric(p, w, st)
         : self   ? launch_pair_prec<kScoreSelf>(p, w, flags, nullptr, st)
                  : launch_pair_prec<kScorePoints>(p, w, flags, shift, st);
    if (rc != SDKDE_OK) return rc;
    if ((rc = profile_mark(0, 1, st)) != SDKDE_OK) return rc;

    const int64_t total = m * (int64_t)d;
    const int nslots = p.sym_on ? p.sym_ngroups + 2 : p.nsplit;
    const int mode = p.thin ? 1 : (self ? 2 : 0);        // see score_epilogue_kernel
    if (!p.thin && epilogue_parts(nslots, total) == kEpiPartsFew) {
        const int64_t quads = m * ((d + 3) / 4);
        constexpr int per_wg = kBlock / kEpiPartsFew;
        if (fused) {
            // plan_fused_prep has checked that this plan and layout are the ones it was made for
            if (!self || !samples_sd_out || p.sym_on || mode != 2) return SDKDE_EINVAL;
            const int blocks_sd = (int)(fused->sd_job.rows_pad / kPrepRows);
            const int blocks_q = (int)(fused->q_job.rows_pad / kPrepRows);
            const auto kernel = format == kFormatHalf2 ? score_epilogue_prep_kernel<true> : score_epilogue_prep_kernel<false>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks_sd + blocks_q)), dim3(kBlock),
                               prep_lds_bytes(p.dp, format), st, w.part_t,
                               w.part_d, w.ps, nslots, m, p.m_pad, d, p.dp, format, inv_ah2, score_out, samples, half_h2,
                               samples_sd_out, quad_io, fused->sd_job, fused->q_job, blocks_sd,
                               w.centre, a, fused->stamp, units);
            return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE;
        }
        const dim3 grid((unsigned)((quads + per_wg - 1) / per_wg));
#define SDKDE_LAUNCH_QUAD(SHIFTED, HALF2)                                                                          \
    hipLaunchKernelGGL((score_epilogue_quad_kernel<SHIFTED, HALF2>), grid, dim3(kBlock), 0, st, w.part_t, w.part_d, w.ps, nslots, m, p.m_pad, d, p.dp, \
                       mode, format, inv_ah2, score_out, samples, half_h2, samples_sd_out, quad_io, least_trusted_sum(n), units, w.part_shift)
        if (w.part_shift) SDKDE_LAUNCH_QUAD(true, true);
        else if (format == kFormatHalf2) SDKDE_LAUNCH_QUAD(false, true);
        else SDKDE_LAUNCH_QUAD(false, false);
#undef SDKDE_LAUNCH_QUAD
    } else {
        SDKDE_LAUNCH_SHIFTED_EPILOGUE(score_epilogue_kernel, w.part_shift, nslots, total, st, w.part_t, w.part_d, w.ps, nslots, m, p.m_pad, d,
                                      p.dp, mode, format, inv_ah2, score_out, samples, half_h2, samples_sd_out, least_trusted_sum(n), units, w.part_shift);
    }
    return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE;
}

// Shared body of sdkde_score and of the first half of sdkde_fit_eval.  samples_sd_out (optional, only at
// the samples themselves): also writes samples + (h^2/2) score from the same epilogue.
int score_impl(const float* samples, int64_t n, const float* points, int64_t m, int32_t d, double h,
               float* score_out, float* samples_sd_out, void* workspace, size_t workspace_bytes, uint32_t flags,
               void* stream, const FusedPrep* fused = nullptr, bool* centre_left = nullptr)
{
    int rc = check_common(samples, n, m, d, h, flags);
    if (rc != SDKDE_OK) return rc;
    const bool self = points == nullptr || (points == samples && m == n);
    if (points == nullptr && m != n) return SDKDE_EINVAL;
    if (m == 0) return SDKDE_OK;
    if (!score_out && !samples_sd_out) return SDKDE_EINVAL;
    if (samples_sd_out && !self) return SDKDE_EINVAL;
    if (!workspace || ((uintptr_t)workspace & 255)) return SDKDE_EWORKSPACE;
    if (flags & SDKDE_FLAG_SAMPLES_PREPARED) return SDKDE_EUNSUPPORTED;      // sdkde_eval / sdkde_eval_laplace only
    flags = two_part_flags(anchored_flags(flags, self), n, d, true, self, workspace_bytes);
    if (fused && fused->whole)
        return score_pass(fused->score_plan, fused->score_at, samples, n, nullptr, m, false, h, score_out, samples_sd_out, flags, (hipStream_t)stream,
                          fused, whole_row_tiles(fused->score_plan, n, m, true, true, false));

    Plan p = make_plan(n, m, d, true, flags);
    apply_symmetric(p, n, flags, self);
    Workspace w;
    int64_t batch = m;
    if (self ? !fit_workspace(p, true, false, workspace, workspace_bytes, flags, &w)
             : (batch = fit_points(p, true, workspace, workspace_bytes, flags, m, &w)) == 0)
        return SDKDE_EWORKSPACE;
    const bool shifted = !self && (flags & SDKDE_FLAG_MAX_SHIFT) != 0;
    if (batch == m && thin_whole(p, n, m, shifted)) {
        // (a workgroup writes while others read the caller's arrays: outputs over them go the other way)
        const size_t in = sizeof(float) * d * n, at_points = sizeof(float) * d * m;
        if (apart(score_out, at_points, samples, in) && apart(samples_sd_out, at_points, samples, in) && apart(score_out, at_points, points, at_points) &&
            apart(score_out, at_points, samples_sd_out, at_points)) {
            const double a = operand_scale(operand_format(p, flags), h);
            const Stamp stamp = make_stamp(w, false, true, samples, n, d, operand_format(p, flags), (float)a, flags);
            if ((rc = profile_mark(0, 0, (hipStream_t)stream)) != SDKDE_OK) return rc;
            rc = launch_thin_whole(samples, n, self ? samples : points, m, d, h, a, score_out, samples_sd_out, stamp, (hipStream_t)stream);
            if (centre_left) *centre_left = false;
            return rc != SDKDE_OK ? rc : profile_mark(0, 1, (hipStream_t)stream);
        }
    }
    int whole_rows = batch == m ? whole_row_tiles(p, n, m, true, self, shifted) : 0;
    if (whole_rows) {
        const Workspace all = whole_layout(p, true, !self, workspace, flags);
        if (all.bytes <= workspace_bytes) w = all;
        else whole_rows = 0;
    }
    for (int64_t first = 0; first < m; first += batch) {
        const int64_t rows = m - first < batch ? m - first : batch;
        if (first > 0) p.row_blocks = (rows + p.rows_per_block - 1) / p.rows_per_block;      // the last batch is shorter
        rc = score_pass(p, w, samples, n, self ? nullptr : points + first * d, rows, first > 0, h,
                        score_out ? score_out + first * d : nullptr, samples_sd_out, flags, (hipStream_t)stream, fused, whole_rows);
        if (rc != SDKDE_OK) return rc;
    }
    return SDKDE_OK;
}

// One pass of an eval call over m queries.  samples_ready: the centre and the prepared samples stand in the workspace, by an
// earlier call (SDKDE_FLAG_SAMPLES_PREPARED) or an earlier pass of this one.  Their place depends on n, d and the precision
// mode only, not on m, and a pass whose record of them does not match gets NaN for every output.
int eval_pass(const Plan& p, const Workspace& w, const float* samples, int64_t n, const float* queries, int64_t m, bool samples_ready,
              double h, float* density_out, float* log_density_out, uint32_t flags, hipStream_t st, bool laplace,
              bool reuse_centre, bool all_prepared, int whole_rows)
{
    int rc;
    const int d = p.d;
    const int format = operand_format(p, flags);
    const double a = operand_scale(format, h);
    const bool shifted = (flags & SDKDE_FLAG_MAX_SHIFT) != 0;
    const PrepJob sample_job{samples, n, p.n_pad, w.xs, nullptr, w.xn, kPadCoord, true, false, half_tail(d, false)};
    const PrepJob query_job{queries, m, p.m_pad, w.ps, nullptr, w.pn, 0.0f, false, shifted, half_tail(d, false)};
    // all_prepared (sdkde_fit_eval): the score epilogue has prepared samples and queries for this plan (plan_fused_prep)
    if (!all_prepared) {
        const Stamp stamp = make_stamp(w, samples_ready, false, samples, n, d, format, (float)a, flags);
        // reuse_centre: w.centre still holds the centre of an earlier pass over (nearly) the same points
        rc = samples_ready ? launch_prep(p, query_job, PrepJob{}, nullptr, 0, a, w, flags, stamp, st)
                           : launch_prep(p, sample_job, query_job, reuse_centre ? nullptr : samples, n, a, w, flags, stamp, st);
        if (rc != SDKDE_OK) return rc;
    }

    const double lognorm = -log((double)n) - (double)d * log(h) - 0.5 * (double)d * log(6.283185307179586476925286766559);
    if ((rc = profile_mark(1, 0, st)) != SDKDE_OK) return rc;
    if (whole_rows) {
        WholeOut out{};
        out.d = d;
        out.min_sum = least_trusted_sum(n);
        out.lognorm = lognorm;
        out.residual = w.residual;
        out.density = density_out;
        out.log_density = log_density_out;
        rc = laplace ? launch_whole<kEvalLaplace>(p, w, whole_rows, m, out, st) : launch_whole<kEval>(p, w, whole_rows, m, out, st);
        return rc != SDKDE_OK ? rc : profile_mark(1, 1, st);
    }
    if (shifted && (rc = launch_max_shift(p, w, flags, st)) != SDKDE_OK) return rc;
    const float* shift = shifted ? w.shift : nullptr;
    rc = laplace ? launch_pair_prec<kEvalLaplace>(p, w, flags, shift, st) : launch_pair_prec<kEval>(p, w, flags, shift, st);
    if (rc != SDKDE_OK) return rc;
    if ((rc = profile_mark(1, 1, st)) != SDKDE_OK) return rc;

    SDKDE_LAUNCH_SHIFTED_EPILOGUE(eval_epilogue_kernel, w.part_shift, p.nsplit, m, st, w.part_d, p.nsplit, m, p.m_pad, lognorm, laplace ? 1 : 0,
                                  w.part_shift ? w.part_shift : shift, w.residual, least_trusted_sum(n), density_out, log_density_out);
    return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE;
}

// Shared body of sdkde_eval and sdkde_eval_laplace.
int eval_impl(const float* samples, int64_t n, const float* queries, int64_t m, int32_t d, double h,
              float* density_out, float* log_density_out, void* workspace, size_t workspace_bytes, uint32_t flags,
              void* stream, bool laplace, bool reuse_centre = false, const FusedPrep* fused = nullptr)
{
    int rc = check_common(samples, n, m, d, h, flags);
    if (rc != SDKDE_OK) return rc;
    if (m == 0) return SDKDE_OK;
    if (!queries || (!density_out && !log_density_out)) return SDKDE_EINVAL;
    if (!workspace || ((uintptr_t)workspace & 255)) return SDKDE_EWORKSPACE;

    flags = two_part_flags(flags, n, d, false, false, workspace_bytes);
    const bool all_prepared = fused != nullptr;
    if (fused && fused->whole)
        return eval_pass(fused->eval_plan, fused->eval_at, samples, n, queries, m, false, h, density_out, log_density_out, flags, (hipStream_t)stream,
                         laplace, reuse_centre, all_prepared, whole_row_tiles(fused->eval_plan, n, m, false, false, false));

    Plan p = make_plan(n, m, d, false, flags);
    Workspace w;
    const int64_t batch = fit_points(p, false, workspace, workspace_bytes, flags, m, &w);
    if (batch == 0) return SDKDE_EWORKSPACE;
    int whole_rows = batch == m ? whole_row_tiles(p, n, m, false, false, (flags & SDKDE_FLAG_MAX_SHIFT) != 0) : 0;
    if (whole_rows) {
        const Workspace all = whole_layout(p, false, true, workspace, flags);
        if (all.bytes <= workspace_bytes) w = all;
        else whole_rows = 0;
    }
    for (int64_t first = 0; first < m; first += batch) {
        const int64_t rows = m - first < batch ? m - first : batch;
        if (first > 0) p.row_blocks = (rows + p.rows_per_block - 1) / p.rows_per_block;      // the last batch is shorter
        rc = eval_pass(p, w, samples, n, queries + first * d, rows, first > 0 || (flags & SDKDE_FLAG_SAMPLES_PREPARED) != 0, h,
                       density_out ? density_out + first : nullptr, log_density_out ? log_density_out + first : nullptr,
                       flags, (hipStream_t)stream, laplace, reuse_centre, all_prepared, whole_rows);
        if (rc != SDKDE_OK) return rc;
    }
    return SDKDE_OK;
}

}  // namespace

// Built-in scratch buffer of sdkde_fit_eval_static: one copy per GPU the library runs on, held until the
// process ends.  The name is a host-side stand-in; the device address is looked up once per device.
static __device__ __align__(256) unsigned char scratch[SDKDE_STATIC_SCRATCH_BYTES];

namespace {

// Address of `scratch` on the current device (resolved on the first call there; null on failure).
void* static_scratch_address()
{
    constexpr int kMaxDevices = 64;
    static std::mutex guard;
    static void* address[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(guard);
    if (!address[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        address[dev] = ptr;
    }
    return address[dev];
}

}  // namespace

extern "C" {

int sdkde_workspace_bytes(int64_t n, int64_t m, int32_t d, uint32_t flags, size_t* bytes)
{
    if (!bytes) return SDKDE_EINVAL;
    int rc = check_common(bytes, n, m, d, 1.0, flags);
    if (rc != SDKDE_OK) return rc;
    *bytes = calls_bytes(n, m, d, flags, true);
    return SDKDE_OK;
}

int sdkde_score(const float* samples, int64_t n, const float* points, int64_t m, int32_t d, double h,
                float* score_out, void* workspace, size_t workspace_bytes, uint32_t flags, void* stream)
{
    if (!score_out && m != 0) return SDKDE_EINVAL;
    return score_impl(samples, n, points, m, d, h, score_out, nullptr, workspace, workspace_bytes, flags, stream);
}

int sdkde_fit_eval(const float* samples, int64_t n, const float* queries, int64_t m, int32_t d, double h,
                   float* score_out, float* samples_sd_out, float* density_out, float* log_density_out,
                   void* workspace, size_t workspace_bytes, uint32_t flags, void* stream)
{
    if (!samples_sd_out) return SDKDE_EINVAL;
    int rc = check_common(samples, n, m, d, h, flags);
    if (rc != SDKDE_OK) return rc;
    if (m > 0 && (!queries || (!density_out && !log_density_out))) return SDKDE_EINVAL;
    if (!workspace || ((uintptr_t)workspace & 255)) return SDKDE_EWORKSPACE;
    // The centre of the samples stays in the workspace; the shifted samples are centred on it too (any
    // centre is exact, it only has to be near the data).  Where the layouts allow it the score epilogue also
    // prepares the eval pass's operands: five launches instead of six, three for small sample sets.
    // Neither where the queries are in an array that the score pass writes: those forms read them before it has.
    FusedPrep fused{};
    const size_t in = sizeof(float) * d * n, at_queries = sizeof(float) * d * m;
    const bool stable = apart(queries, at_queries, samples_sd_out, in) && apart(queries, at_queries, score_out, in);
    const bool fuse = stable && plan_fit(samples_sd_out, n, queries, m, d, h, workspace, workspace_bytes, flags, &fused);
    bool centre_left = true;
    rc = score_impl(samples, n, nullptr, n, d, h, score_out, samples_sd_out, workspace, workspace_bytes, flags, stream, fuse ? &fused : nullptr, &centre_left);
    if (rc != SDKDE_OK || m == 0) return rc;
    return eval_impl(samples_sd_out, n, queries, m, d, h, density_out, log_density_out, workspace, workspace_bytes,
                     flags, stream, false, centre_left, fuse ? &fused : nullptr);
}

int sdkde_fit_eval_static(const float* samples, int64_t n, const float* queries, int64_t m, int32_t d, double h,
                          float* score_out, float* samples_sd_out, float* density_out, float* log_density_out,
                          uint32_t flags, void* stream)
{
    if (!samples_sd_out) return SDKDE_EINVAL;
    int rc = check_common(samples, n, m, d, h, flags);
    if (rc != SDKDE_OK) return rc;
    // The pass takes the decomposition the ordinary call would take, so that both give the same bits, where the built-in
    // buffer holds a workspace of sdkde_workspace_bytes.  A pass that needs more is served on the fp32 mode's operands
    // while both of its steps fit with fewer splits or the queries in batches, and refused before anything is launched
    // otherwise.
    Plan score_plan = make_plan(n, n, d, true, flags), eval_plan = make_plan(n, m, d, false, flags);
    apply_symmetric(score_plan, n, flags, true);
    Workspace unused;
    if (!score_plan.parts && !eval_plan.parts && calls_bytes(n, m, d, flags, false) > (size_t)SDKDE_STATIC_SCRATCH_BYTES) return SDKDE_ETOOLARGE;
    if (!fit_workspace(score_plan, true, false, nullptr, SDKDE_STATIC_SCRATCH_BYTES, flags, &unused) ||
        (m > 0 && !fit_points(eval_plan, false, nullptr, SDKDE_STATIC_SCRATCH_BYTES, flags, m, &unused)))
        return SDKDE_ETOOLARGE;
    void* ws = static_scratch_address();
    if (!ws) return SDKDE_EDEVICE;
    return sdkde_fit_eval(samples, n, queries, m, d, h, score_out, samples_sd_out, density_out, log_density_out, ws,
                          (size_t)SDKDE_STATIC_SCRATCH_BYTES, flags, stream);
}

int sdkde_debias(const float* samples, const float* score, int64_t n, int32_t d, double h, float* samples_sd_out,
                 void* stream)
{
    if (!samples || !score || !samples_sd_out || n < 0 || d < 1 || bad_bandwidth(h)) return SDKDE_EINVAL;
    const int64_t total = n * (int64_t)d;
    if (total == 0) return SDKDE_OK;
    hipLaunchKernelGGL(debias_kernel, dim3((unsigned)((total + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                       (hipStream_t)stream, samples, score, total, (float)(0.5 * h * h), samples_sd_out);
    return hipGetLastError() == hipSuccess ? SDKDE_OK : SDKDE_EDEVICE;
}

int sdkde_eval(const float* samples_sd, int64_t n, const float* queries, int64_t m, int32_t d, double h,
               float* density_out, float* log_density_out, void* workspace, size_t workspace_bytes, uint32_t flags,
               void* stream)
{
    return eval_impl(samples_sd, n, queries, m, d, h, density_out, log_density_out, workspace, workspace_bytes, flags,
                     stream, false);
}

int sdkde_eval_laplace(const float* samples, int64_t n, const float* queries, int64_t m, int32_t d, double h,
                       float* density_out, void* workspace, size_t workspace_bytes, uint32_t flags, void* stream)
{
    return eval_impl(samples, n, queries, m, d, h, density_out, nullptr, workspace, workspace_bytes, flags, stream,
                     true);
}

int sdkde_describe_plan(int64_t n, int64_t m, int32_t d, int32_t call, uint32_t flags, int64_t* out, int32_t out_len)
{
    if (!out || out_len < 20 || call < 0 || call > 2) return SDKDE_EINVAL;
    int rc = check_common(out, n, m, d, 1.0, flags);
    if (rc != SDKDE_OK) return rc;
    const bool score = call != 2;
    const bool separate = call != 0;
    const int64_t rows = call == 0 ? n : m;
    if (score) flags = anchored_flags(flags, !separate);
    Plan p = make_plan(n, rows, d, score, flags);
    if (score) apply_symmetric(p, n, flags, !separate);
    char* const base = reinterpret_cast<char*>(uintptr_t(1) << 20);      // any aligned non-null address: offsets only
    const Workspace w = layout(p, score, separate, base, flags);
    auto off = [&](const void* q) { return q ? (int64_t)((const char*)q - base) : (int64_t)-1; };
    const int64_t slots = p.sym_on ? p.sym_ngroups + 2 : p.nsplit;
    const int64_t xt_scale = effective_prec(flags, p.thin, p.dp) == SDKDE_PREC_FP16X2_ALL ? 2 : 1;
    const int64_t v[20] = {
        p.thin ? 1 : 0, p.dp, p.ni, p.rows_per_block, p.row_blocks, p.nsplit, p.tiles_per_split, p.ntiles,
        p.n_pad, p.m_pad, (int64_t)w.bytes, off(w.xs), off(w.xt), off(w.xn), off(w.ps), off(w.pn),
        off(w.part_t), off(w.part_d), slots, xt_scale};
    for (int k = 0; k < 20; ++k) out[k] = v[k];
    if (out_len >= 24) {
        out[20] = p.sym_on ? 1 : 0;
        out[21] = p.sym_on ? p.sym_rb : 0;
        out[22] = p.sym_on ? p.sym_per_group : 0;
        out[23] = p.sym_on ? p.sym_ngroups : 0;
    }
    if (out_len >= 25) out[24] = 4;
    if (out_len >= 26) {
        out[25] = 0;
        size_t need = 0;
        FusedPrep unused;
        if (call == 2 && sdkde_workspace_bytes(n, m, d, flags, &need) == SDKDE_OK)
            out[25] = plan_fused_prep(nullptr, n, nullptr, m, d, 1.0, base, need, anchored_flags(flags, true), flags, &unused) ? 1 : 0;
    }
    return SDKDE_OK;
}

int sdkde_set_tuning(int knob, int value)
{
    if (knob < 0 || knob >= SDKDE_TUNE_COUNT || value < 0) return SDKDE_EINVAL;
    g_tuning[knob].store(value, std::memory_order_relaxed);
    return SDKDE_OK;
}

const char* sdkde_status_string(int status)
{
    switch (status) {
        case SDKDE_OK: return "ok";
        case SDKDE_EINVAL: return "invalid argument";
        case SDKDE_EUNSUPPORTED: return "unsupported dimension, size or flag";
        case SDKDE_EWORKSPACE: return "workspace missing, misaligned or too small";
        case SDKDE_EDEVICE: return "HIP runtime error";
        case SDKDE_ETOOLARGE: return "problem too large for the built-in scratch buffer";
        default: return "unknown status";
    }
}

int sdkde_profile_enable(int on)
{
    g_profile.enabled = on != 0;
    g_profile.count[0] = g_profile.count[1] = 0;
    return SDKDE_OK;
}

int sdkde_profile_summary(int which, int* launches, float* total_ms)
{
    if (which < 0 || which > 1 || !launches || !total_ms) return SDKDE_EINVAL;
    float total = 0.0f;
    for (int k = 0; k < g_profile.count[which]; ++k) {
        float ms = 0.0f;
        SDKDE_HIP(hipEventSynchronize(g_profile.ev[which][k][1]));
        SDKDE_HIP(hipEventElapsedTime(&ms, g_profile.ev[which][k][0], g_profile.ev[which][k][1]));
        total += ms;
    }
    *launches = g_profile.count[which];
    *total_ms = total;
    return SDKDE_OK;
}

}  // extern "C"
