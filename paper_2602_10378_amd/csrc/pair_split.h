// Pair kernel of the fp32 matrix path (d >= 4): both contractions on the bf16 matrix units over three-part operands.
#pragma once
#include "common.h"
#include "split3.h"

namespace {

// ------------------------------------------------------------------------------------------
// A wave owns NI tiles of 16 evaluation rows (their parts in registers, the B operand) and walks over chunks of 32
// samples (two 16-sample tiles) that the WAVES waves of the workgroup share through LDS.  Per (row tile, chunk):
//   C[j][i] = -|p_i|^2/2 - |x_j|^2/2 + x_j . p_i   6 KB v_mfma_f32_16x16x32_bf16 (3 KB per sample tile, fp32 accumulate)
//   Phi     = exp2(C), D_i += sum_j Phi            fp32 VALU
//   T^T    += X_J^T Phi^T                          6 KB MFMAs over the 32 samples (SCORE only), Phi split in registers
// The 16x16 accumulator layout (lane (r, g), register v) = (sample 4g + v, row r) is the B operand layout (k = 8g + e,
// column r) of the second contraction for the samples {4g + e of tile 0, 4g + e - 4 of tile 1}, the order in which the
// prepared transpose stores them: Phi never leaves its lane.
//
// What bounds it: on this chip the bf16 MFMA (16 clocks; about 21 when every SIMD issues nothing else, the clock then
// drops under the power limit) and the vector instructions of a SIMD overlap by little, so the time is close to the
// sum of both: per 256 pairs 3 KB MFMAs for each contraction, 4 v_exp_f32 at 8 clocks, 24 + 2 KB (eval: 8) adds, subtracts
// and ands at about 2.4 and (score) 6 v_perm_b32 at 4.6.  That sum is 218 clocks for the score at dp = 16 (fp32 MFMA kernel
// before: 333) and 52 + 48 KB for eval; measured figures at the dispatch (split_shape in sdkde.hip).  Two waves per SIMD are needed (one wave:
// 1238 clocks against 983 at dp = 96) and more do not help; NI row tiles share every operand read from LDS.
//
// SELF (score at the samples themselves): the pair (i, i) must stay out of D and T, because T_i/D_i - x_i would
// otherwise cancel against the large self term whenever a point has few neighbours; the epilogue restores it
// analytically (phi_ii = 1).  In the chunks that are a wave's own rows a wave-uniform branch sets the diagonal's exponents to
// -3e38 between the Gram MFMAs and the exponentials (a masked copy of the whole body in the loop spills; going over those
// chunks after the loop, from global memory, kept the workgroups they fall to longer).
//
// Grid: blockIdx.x = row_block * S + split; each workgroup handles 16 NI WAVES rows and the sample tiles
// [split*tiles_per_split, min(ntiles, (split+1)*tiles_per_split)).  With S a multiple of 8 the round-robin placement of
// workgroups on the 8 XCDs makes each XCD stream only its own eighth of the samples through its L2.
// ntiles and tiles_per_split are even (host side); ps, pn hold m_pad rows, xs, xt, xn ntiles * 16 rows.
// ------------------------------------------------------------------------------------------

// Row-tile operands of one wave: -|p~|^2/2 and the parts of p~ as the lane's 16 bytes of each B operand.
// FOUR (KB = 1, d <= 4): the six part products of four columns fill 24 of the 32 of one operand, four columns each:
// [h h | m m | h l | -] against [h m | h m | l h | 0].
template <int KB, int NI, bool FOUR = false>
struct SplitRows {
    static constexpr int PAIRS = KB / 2;        // 32-column blocks
    static constexpr bool ODD = KB % 2 != 0;    // and a 16-column one
    bf16x8 b[NI][PAIRS > 0 ? PAIRS : 1][3];     // h, m, l
    bf16x8 o[ODD ? NI : 1][2];                  // K = 32 as two parts of 16 columns: [h | m] and [l | h]
    float ni[NI];

    __device__ __forceinline__ void load(const float* __restrict__ ps, const float* __restrict__ pn, int64_t row0, int r, int g)
    {
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const char* tile = reinterpret_cast<const char*>(ps) + (row0 / kTile + t) * (int64_t)(KB * 1536);
#pragma unroll
            for (int p = 0; p < PAIRS; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    b[t][p][q] = *reinterpret_cast<const bf16x8*>(tile + p * 3072 + q * kPartBytes + (16 * g + r) * 16);
            if (FOUR) {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const char* base = tile + r * 16;
                const u32x2 lo = *reinterpret_cast<const u32x2*>(base + (g == 2 ? 1024 : 0));
                const u32x2 hi = *reinterpret_cast<const u32x2*>(base + (g < 2 ? 512 : 0));
                const u32x4 both = g == 3 ? u32x4{0, 0, 0, 0} : u32x4{lo.x, lo.y, hi.x, hi.y};
                o[t][0] = __builtin_bit_cast(bf16x8, both);
            } else if (ODD) {
                const char* base = tile + PAIRS * 3072 + (16 * (g & 1) + r) * 16;
                o[t][0] = *reinterpret_cast<const bf16x8*>(base + (g < 2 ? 0 : 512));
                o[t][1] = *reinterpret_cast<const bf16x8*>(base + (g < 2 ? 1024 : 0));
            }
            ni[t] = pn[row0 + t * kTile + r];
        }
    }
};

// Where the second-level sums of T live: at dp <= 64 in LDS (registers are what two waves per SIMD leave short), above
// in the wave's own rows of its partial slot (LDS is full of samples there): read, added to and written once per
// kFlushTiles sample tiles.
constexpr bool split_sums_in_lds(int kb) { return kb <= 4; }

// NB: row tiles whose Gram accumulators and split weights are live at a time.  AHEAD: operands are read from LDS a whole
// group of MFMAs before their use.
template <int KB, int NI, int WAVES, int NB, bool AHEAD, int MINW, int KIND>
__global__ __launch_bounds__(WAVES * kWave, MINW) void pair_split_kernel(
    const float* __restrict__ ps, const float* __restrict__ pn, const float* __restrict__ xs,
    const float* __restrict__ xt, const float* __restrict__ xn, float* __restrict__ part_t,
    float* __restrict__ part_d, int ntiles, int tiles_per_split, int nsplit, int64_t m_pad, float laplace_c0,
    const float* __restrict__ shift)
{
    static_assert(NI % 2 == 0 && NI % NB == 0, "a wave's own rows are whole chunks");
    constexpr bool BAND = KIND == kScoreBand;
    constexpr bool SCORE = KIND == kScoreSelf || KIND == kScorePoints || BAND;
    constexpr bool SELF = KIND == kScoreSelf || BAND;
    constexpr bool LAPLACE = KIND == kEvalLaplace;
    constexpr bool FOUR = KIND == kRowMaxFour;                   // see SplitRows
    constexpr bool ROWMAX = KIND == kRowMax || FOUR;
    static_assert(!FOUR || (KB == 1 && !AHEAD), "four columns: one operand, read where it is used");
    constexpr int DP = KB * 16;
    constexpr int KT = SCORE ? KB : 1;
    constexpr int PAIRS = KB / 2;
    constexpr bool ODD = KB % 2 != 0;
    constexpr int XCH = 3 * KB;                                  // 1 KiB pieces of a chunk of xs (and of xt)
    constexpr int CH = SCORE ? 2 * XCH : XCH;
    constexpr int STAGE = (CH + WAVES - 1) / WAVES;              // pieces a wave moves per chunk
    constexpr bool SUMLDS = SCORE && split_sums_in_lds(KB);
    __shared__ __align__(16) char stage_lds[2][CH * kPartBytes];
    __shared__ f32x4 sum_lds[SUMLDS ? WAVES : 1][SUMLDS ? NI * KT : 1][SUMLDS ? kWave : 1];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);    // wave-uniform by construction
    const int r = lane & 15, g = lane >> 4;
    const int split = blockIdx.x % nsplit;
    const int64_t row_block = blockIdx.x / nsplit;
    const int64_t row0 = (row_block * WAVES + wave) * (NI * kTile);

    SplitRows<KB, NI, FOUR> rows;
    rows.load(ps, pn, row0, r, g);

    // Two-level accumulation: the running sums (tacc, dacc) are folded into a second level every kFlushTiles sample
    // tiles, so no fp32 accumulator sees more than a short chain of additions at its own magnitude.
    f32x4 tacc[NI][KT];
    float dacc[NI], dsum[NI];
    float lc0[LAPLACE ? NI : 1];          // Laplace factor constant per row tile: 1 + d/2 + shift_i ln 2
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        dacc[t] = dsum[t] = ROWMAX ? kNegHuge : 0.0f;
#pragma unroll
        for (int mb = 0; mb < KT; ++mb) {
            tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (SUMLDS) sum_lds[wave][t * KT + mb][lane] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (LAPLACE) lc0[t] = fmaf(shift ? shift[row0 + t * kTile + r] : 0.0f, kLn2, laplace_c0);
    }
    auto slot_at = [&](int t, int mb) {
        return reinterpret_cast<f32x4*>(part_t + ((int64_t)split * m_pad + row0 + t * kTile + r) * DP + g * 4 + mb * 16);
    };

    // One chunk against all NI row tiles.  own (SELF): the row tile that is the chunk's first sample tile, if it is one.
    auto chunk = [&](const char* xc, const char* tc, const f32x4& nj0, const f32x4& nj1, int own) {
        constexpr int GROUPS = PAIRS + (ODD ? 1 : 0);
        constexpr int STEPS = 2 * GROUPS - 1;      // leading products of all groups but the last, the last, the others' rest
        // Operands of one group of MFMAs; scheduling barriers keep an early read early.
        bf16x8 ga[2][2][3], ta[2][3];
        auto pin = [] { if (AHEAD) __builtin_amdgcn_sched_barrier(0); };
        auto read_gram = [&](int s, bf16x8 (&a)[2][3]) {
            if (GROUPS == 2 && s == GROUPS) return;             // still there from the first step
            const int p = s < GROUPS ? s : s - GROUPS;
            const int parts = GROUPS > 2 && s < GROUPS - 1 ? 1 : 3;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const char* base = xc + u * (KB * 1536) + p * 3072;
                if (p < PAIRS) {
#pragma unroll
                    for (int q = 0; q < parts; ++q) a[u][q] = *reinterpret_cast<const bf16x8*>(base + q * kPartBytes + lane * 16);
                } else if (FOUR) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    const char* row = base + r * 16;
                    const u32x2 lo = *reinterpret_cast<const u32x2*>(row + (g == 1 ? 512 : 0));
                    const u32x2 hi = *reinterpret_cast<const u32x2*>(row + (g == 1 ? 512 : g == 2 ? 1024 : 0));
                    a[u][0] = __builtin_bit_cast(bf16x8, (u32x4){lo.x, lo.y, hi.x, hi.y});
                } else {                            // [h | h], [m | m], [h | l]
                    const char* half = base + (16 * (g & 1) + r) * 16;
                    a[u][0] = *reinterpret_cast<const bf16x8*>(half);
                    a[u][1] = *reinterpret_cast<const bf16x8*>(half + 512);
                    a[u][2] = *reinterpret_cast<const bf16x8*>(half + (g < 2 ? 0 : 1024));
                }
            }
        };
        auto read_t = [&](int mb, bf16x8 (&a)[3]) {
#pragma unroll
            for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const bf16x8*>(tc + mb * 3072 + q * kPartBytes + lane * 16);
        };
#pragma unroll
        for (int t0 = 0; t0 < NI; t0 += NB) {
            f32x4 c[NB][2];
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                c[t][0] = nj0 + rows.ni[t0 + t];
                c[t][1] = nj1 + rows.ni[t0 + t];
            }
            if (AHEAD) read_gram(0, ga[0]);
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                if (!AHEAD) read_gram(s, ga[s & 1]);
                else if (s + 1 < STEPS) read_gram(s + 1, ga[(s + 1) & 1]);
                else if (SCORE) read_t(0, ta[0]);
                pin();
                const bf16x8 (&a)[2][3] = ga[s & 1];
                // the largest products of all groups first: they bring the accumulator from the size of the norms down
                // to that of the distance, where the small ones round finer (error of the score against 64 bits, fp32
                // MFMAs / this order: d = 64 1.3e-6 / 1.1e-6, d = 90 2.7e-6 / 1.9e-6, d = 128 3.4e-6 / 2.5e-6)
                const int p = s < GROUPS ? s : s - GROUPS;
                const int k0 = s < GROUPS ? 0 : 1, k1 = s < GROUPS - 1 ? 1 : 6;
                if (p < PAIRS) {
                    constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
                    for (int k = k0; k < k1; ++k)
#pragma unroll
                        for (int t = 0; t < NB; ++t)
#pragma unroll
                            for (int u = 0; u < 2; ++u)
                                c[t][u] = mfma_bf16(a[u][PA[k]], rows.b[t0 + t][p < PAIRS ? p : 0][PB[k]], c[t][u]);
                } else {
                    // [h | h] [h | m], [m | m] [h | m], [h | l] [l | h]
#pragma unroll
                    for (int k = 0; k < (FOUR ? 1 : 3); ++k)
#pragma unroll
                        for (int t = 0; t < NB; ++t)
#pragma unroll
                            for (int u = 0; u < 2; ++u)
                                c[t][u] = mfma_bf16(a[u][k], rows.o[ODD ? t0 + t : 0][k == 2 ? 1 : 0], c[t][u]);
                }
                pin();
            }
            if (SELF && (unsigned)own < (unsigned)NI) {         // wave-uniform: the pairs of a point with itself
#pragma unroll
                for (int t = 0; t < NB; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (own + u == t0 + t) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) c[t][u][v] = g * 4 + v == r ? kNegHuge : c[t][u][v];
                        }
            }
            bf16x8 w[NB][3];
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                float& dt = dacc[t0 + t];
                if (ROWMAX) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) dt = fmaxf(dt, fmaxf(fmaxf(c[t][u].x, c[t][u].y), fmaxf(c[t][u].z, c[t][u].w)));
                    continue;
                }
                f32x4 phi[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) phi[u][v] = __builtin_amdgcn_exp2f(c[t][u][v]);
                    if (LAPLACE) {
                        // c is the base-2 exponent -r^2/(2h^2) log2(e) (less the row's shift), so the Laplace factor
                        // 1 + d/2 - r^2/(2h^2) is lc0 + c ln 2 (Laplace-corrected KDE section)
#pragma unroll
                        for (int v = 0; v < 4; ++v) dt = fmaf(phi[u][v], fmaf(c[t][u][v], kLn2, lc0[t0 + t]), dt);
                    } else {
                        dt += (phi[u].x + phi[u].y) + (phi[u].z + phi[u].w);
                    }
                }
                // keeps the sum here: the compiler would otherwise sink it behind the MFMAs and hold the Phi tiles live
                if (SCORE) asm volatile("" : "+v"(dt));
                if (SCORE) split3_weights(phi[0], phi[1], w[t][0], w[t][1], w[t][2]);
            }
            if constexpr (SCORE) {
                f32x4 sum[2][NB];
                auto add = [&](int mb) {
#pragma unroll
                    for (int t = 0; t < NB; ++t) tacc[t0 + t][mb] += sum[mb & 1][t];
                };
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) {
                    if (!AHEAD) read_t(mb, ta[mb & 1]);
                    else if (mb + 1 < KB) read_t(mb + 1, ta[(mb + 1) & 1]);
                    pin();
                    const bf16x8 (&a)[3] = ta[mb & 1];
                    // The chunk's sum starts from zero, its smallest products first: an MFMA rounds its accumulator after
                    // every lane group (four times), which this way happens at the size of 32 terms and not of the
                    // running sum (summing into tacc directly: score error 1.0e-6 against 3.7e-7 at n = 32768, d = 16).
                    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
                    for (int k = 0; k < 6; ++k)
#pragma unroll
                        for (int t = 0; t < NB; ++t)
                            sum[mb & 1][t] = mfma_bf16(a[PA[k]], w[t][PB[k]], k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[mb & 1][t]);
                    pin();
                    // added a group later, when the MFMAs have finished
                    if (mb > 0) add(mb - 1);
                }
                add(KB - 1);
            }
        }
    };

    const int own0 = (int)(row0 / kChunkRows);              // SELF: the wave's own rows are chunks own0 .. own0 + NI/2 - 1
    // BAND (the symmetric mode's in-block pass): only the samples of the rows' own block, tiles_per_split tiles long and a
    // multiple of the workgroup's rows; nsplit is 1.
    const int first_tile = BAND ? (int)(row_block * (WAVES * NI) / tiles_per_split) * tiles_per_split : split * tiles_per_split;
    const int c_begin = first_tile / 2;
    const int c_end = min(ntiles, first_tile + tiles_per_split) / 2;
    const char* const xs_b = reinterpret_cast<const char*>(xs);
    const char* const xt_b = reinterpret_cast<const char*>(xt);
    bool flushed = false;                                   // !SUMLDS: the partial slot holds second-level sums
    if (c_begin < c_end) {
        const int c_last = c_end - 1;                       // the prefetch past the end re-reads the last chunk (in bounds)
        // The pieces a wave moves: both arrays advance by the same bytes per chunk, so one scalar base each (no branches
        // in the loop).  A piece past the end is the last one again, deposited twice with the same bytes.
        auto piece_of = [&](int q) { return (q + 1) * WAVES <= CH ? q * WAVES + wave : min(q * WAVES + wave, CH - 1); };
        const char* src[STAGE];
#pragma unroll
        for (int q = 0; q < STAGE; ++q) {
            const int piece = piece_of(q);                                  // wave-uniform
            src[q] = !SCORE || piece < XCH ? xs_b + piece * kPartBytes : xt_b + (piece - XCH) * kPartBytes;
        }
        f32x4 stage[STAGE];
        auto fetch = [&](int c) {
            const int64_t at = (int64_t)min(c, c_last) * (XCH * kPartBytes);
#pragma unroll
            for (int q = 0; q < STAGE; ++q) stage[q] = *reinterpret_cast<const f32x4*>(src[q] + at + lane * 16);
        };
        auto deposit = [&](char* buf) {
#pragma unroll
            for (int q = 0; q < STAGE; ++q) *reinterpret_cast<f32x4*>(buf + piece_of(q) * kPartBytes + lane * 16) = stage[q];
        };
        auto norms = [&](int c, int u) {
            return *reinterpret_cast<const f32x4*>(xn + (int64_t)min(c, c_last) * kChunkRows + u * kTile + g * 4);
        };
        f32x4 nj0 = norms(c_begin, 0), nj1 = norms(c_begin, 1);
        fetch(c_begin);
        deposit(stage_lds[0]);
        __syncthreads();
        for (int c = c_begin; c < c_end; ++c) {             // the same bounds for all waves of the workgroup
            const char* cur = stage_lds[(c - c_begin) & 1];
            fetch(c + 1);                                   // lands in registers while this chunk is worked on
            const f32x4 nn0 = norms(c + 1, 0), nn1 = norms(c + 1, 1);
            chunk(cur, cur + XCH * kPartBytes, nj0, nj1, 2 * (c - own0));
            if (!ROWMAX && ((c + 1 - c_begin) & (kFlushTiles / 2 - 1)) == 0) {
#pragma unroll
                for (int t = 0; t < NI; ++t) {
                    dsum[t] += dacc[t];
                    dacc[t] = 0.0f;
                    if constexpr (SCORE) {
#pragma unroll
                        for (int mb = 0; mb < KT; ++mb) {
                            f32x4* const at = SUMLDS ? &sum_lds[wave][t * KT + mb][lane] : slot_at(t, mb);
                            *at = SUMLDS || flushed ? *at + tacc[t][mb] : tacc[t][mb];
                            tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
                    }
                }
                flushed = true;
            }
            nj0 = nn0;
            nj1 = nn1;
            // The other buffer was last read before the previous barrier; this barrier publishes the new chunk and
            // ends the reads of the current one.
            deposit(stage_lds[(c + 1 - c_begin) & 1]);
            __syncthreads();
        }
    }
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        if constexpr (SCORE) {
#pragma unroll
            for (int mb = 0; mb < KT; ++mb) {
                if (SUMLDS) tacc[t][mb] += sum_lds[wave][t * KT + mb][lane];
                else if (flushed) tacc[t][mb] += *slot_at(t, mb);
                *slot_at(t, mb) = tacc[t][mb];
            }
        }
        // D needs the sum (or maximum) over the four lane groups g
        float dtot = ROWMAX ? fmaxf(dsum[t], dacc[t]) : dsum[t] + dacc[t];
#pragma unroll
        for (int step = 16; step <= 32; step *= 2) {
            const float other = __shfl_xor(dtot, step);
            dtot = ROWMAX ? fmaxf(dtot, other) : dtot + other;
        }
        if (g == 0) part_d[(int64_t)split * m_pad + row0 + t * kTile + r] = dtot;
    }
}

}  // namespace
