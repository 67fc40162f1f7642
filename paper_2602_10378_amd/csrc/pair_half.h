// Pair kernel of the fp32 matrix path (d >= 4): both contractions on the fp16 matrix units over two-part operands.
//
// What bounds it: instruction issue, under the card's power limit.  Busy with MFMAs and exps the clock settles at 1.9 to 2.3 of
// its 2.4 GHz; prefetching deeper, interleaving the MFMAs of one row tile with the vector work of another and cheaper barriers
// changed no time, only fewer instructions do.  Three-part bf16 operands, which this replaces, took six MFMAs per product where
// two fp16 parts take three, twice the Gram operands in registers and LDS, and four vector instructions a weight and part.
// What an fp16 part lacks is range, hence the row scale of the weights (set_scale) and the scaled rows of distant points (half2.h).
// Clocks of a wave's 16 x 16 pairs at 2.4 GHz, four SIMDs full, before / now:
//   eval  d = 16 107 / 75 (d <= 8: 63), d = 32 161 / 110, d = 64 280 / 176, d = 128 646 / 326
//   score d = 16 234 / 178 (d <= 8: 155), d = 32 344 / 252, d = 48 529 / 354, d = 64 634 / 462, d = 96 983 / 695, d = 128 1550 / 890
// Whole calls: score + eval at 32768 samples, d = 16, 641 / 484 us; 262144 x 65536, d = 64, 79.7 / 53.8 ms; eval of 1024 points
// against 1048576 samples, d = 16, 217 / 155 us.  Error against 64-bit sums over d = 4 .. 128, geometric mean of now / before:
// score 0.85 (at most 1.07), at separate points 0.94 (1.08), density 0.86, Laplace-corrected 0.67.
//
// Max-shifted sums (FAR) find the shift as they go: a row's is set from its largest exponent in a split's first chunk and raised
// when a weight outgrows what its sums hold (2^100 for the eval kinds, so hardly ever), and each slot keeps its own for the
// epilogue to add the slots with.  A first pass over all samples for the row maxima, on the leading products, and a launch that put them
// into the norms came before; two passes / one: eval 50021 x 10007, d = 24, 155 / 110 us, 20000 x 5003, d = 16 50 / 36, d = 128 136 / 93;
// Laplace 100000 x 20000, d = 32, 659 / 493; score at points 20000 x 20000, d = 16 229 / 155, d = 64 441 / 343, 20000 x 5003,
// d = 128 299 / 289 (its rows' scales are raised often).  Errors against 64-bit sums as before (0.97 to 1.02).
#pragma once
#include "common.h"
#include "half2.h"
#include "split3.h"

namespace {

// Row-tile operands of one wave: the parts of p~ as the lane's 16 bytes of each B operand, and the rows' constant terms.
template <int KB, int TAIL, int NI, bool SCORE, bool FAR>
struct HalfRows {
    static constexpr int PAIRS = KB / 2;            // 32-column blocks
    static constexpr bool ODD = TAIL == kTailSixteen || TAIL == kTailEight, SPARE = TAIL == kTailSpare;
    static constexpr int TERM = TAIL == kTailSixteen ? 1 : 0;           // operand and lane group that hold the term
    static constexpr int TERM_GROUP = TAIL == kTailSixteen ? 2 : 3;
    f16x8 b[NI][PAIRS > 0 ? PAIRS : 1][2];          // h, l
    // 16 columns: [h | h], [l | term, residual factor, l of four columns, l of eight]; 8 columns: [h, l, h, as before]
    f16x8 o[ODD ? NI : 1][TAIL == kTailSixteen ? 2 : 1];
    float term[NI];

    __device__ __forceinline__ void load(const float* __restrict__ ps, const float* __restrict__ pn, int64_t row0, int r, int g)
    {
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const char* tile = reinterpret_cast<const char*>(ps) + (row0 / kTile + t) * (int64_t)half_tile_bytes(KB);
#pragma unroll
            for (int p = 0; p < PAIRS; ++p)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    b[t][p][q] = *reinterpret_cast<const f16x8*>(tile + p * 2048 + q * 1024 + (16 * g + r) * 16);
            const char* base = tile + PAIRS * 2048 + r * 16;
            if constexpr (TAIL == kTailSixteen) {
                o[t][0] = *reinterpret_cast<const f16x8*>(base + (g & 1) * 256);
                o[t][1] = *reinterpret_cast<const f16x8*>(base + 512 + (g == 1 || g == 2 ? 256 : 0));
            } else if constexpr (TAIL == kTailEight) {
                o[t][0] = *reinterpret_cast<const f16x8*>(base + (g == 1 || g == 3 ? 512 : 0));
            }
            if (ODD && g == TERM_GROUP) {
                f16x8& e = o[t][TERM];
                // the eval kinds' term is not lowered by a scale and as large as the norms: beside it, what an MFMA truncates of
                // the small products of its lane group would cost more than they give, and all one way (density at n = 4096,
                // d = 16: error 4.9e-7 with them, 3.2e-7 without)
                e = SCORE ? f16x8{0, 0, 0, (_Float16)kResidualFactor, e[0], e[1], e[2], e[3]} : f16x8{0, 0, 0, 0, 0, 0, 0, 0};
            }
            if (SPARE && g == TERM_GROUP) b[t][SPARE ? PAIRS - 1 : 0][0] = f16x8{0, 0, 0, SCORE ? (_Float16)kResidualFactor : (_Float16)0, 0, 0, 0, 0};
            term[t] = pn[row0 + t * kTile + r];
        }
    }
    // What rounding the row's norm left, from its prepared row.
    __device__ __forceinline__ float residual(const float* __restrict__ ps, int64_t row) const
    {
        if (TAIL == kTailNone) return 0.0f;
        const char* tile = reinterpret_cast<const char*>(ps) + row / kTile * (int64_t)half_tile_bytes(KB);
        const char* at = SPARE ? tile + (PAIRS - 1) * 2048 + TERM_GROUP * 256 : tile + PAIRS * 2048 + 1024;
        return (float)reinterpret_cast<const _Float16*>(at + row % kTile * 16)[3] * kResidualFactor;
    }
    // Products as the eval kinds have them.
    __device__ __forceinline__ void bare(int g)
    {
#pragma unroll
        for (int t = 0; t < NI; ++t)
            if (g == TERM_GROUP) {
                if (ODD) o[ODD ? t : 0][TERM] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
                if (SPARE) b[t][SPARE ? PAIRS - 1 : 0][0] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
            }
    }
    // The row's term in the spare columns of the last operand.
    __device__ __forceinline__ void place_term(int t, float v, float residual, int g)
    {
        if (TAIL == kTailNone) return;
        _Float16 part[3];
        split_term<FAR>(v, residual, part);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            f16x8& e = ODD ? o[ODD ? t : 0][TERM] : b[t][SPARE ? PAIRS - 1 : 0][0];
            e[q] = g == TERM_GROUP ? part[q] : e[q];
        }
    }
};

// Weights are formed as 2^kWeightScale times what goes into the sums' first part, so that the second part, which is the rest of
// the division by 2^kWeightScale, comes out in a range of its own: with W = 2^11 w, h = fp16(w), l = fp16(W - 2^11 h), and l
// meets the transposed samples' third part, 2^-11 h.  Where the first part alone would be below the fp16 range the second still
// holds 11 bits down to 2^-25 of a W of one.
constexpr float kMostWeight = 65000.0f * kWeightScale;      // of a lane's sum of W of a row, so that no w leaves the fp16 range
constexpr int kRaisedTo = 18;                       // where a row's largest W is put when it has outgrown that
constexpr float kLeastShift = -126.0f;              // a W of one then stands for the smallest normal fp32 number
// Shifted sums without Phi X have the fp32 range for their weights: a row's first look puts its largest at one.
constexpr float kMostShifted = 1.0e30f;             // of a lane's sum over the row tiles at hand

__device__ __forceinline__ void split_weights(const f32x4& p, const f32x4& q, f16x8& h, f16x8& l)
{
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    uint32_t hw[4], lw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float a = k < 2 ? p[2 * k] : q[2 * k - 4], b = k < 2 ? p[2 * k + 1] : q[2 * k - 3];
        const f16x2 hh = __builtin_convertvector((f32x2{a * (1.0f / kWeightScale), b * (1.0f / kWeightScale)}), f16x2);
        const f32x2 rest = {fmaf((float)hh.x, -kWeightScale, a), fmaf((float)hh.y, -kWeightScale, b)};
        hw[k] = __builtin_bit_cast(uint32_t, hh);
        lw[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, f16x2));
    }
    h = __builtin_bit_cast(f16x8, (u32x4){hw[0], hw[1], hw[2], hw[3]});
    l = __builtin_bit_cast(f16x8, (u32x4){lw[0], lw[1], lw[2], lw[3]});
}

// Where the second-level sums of T live: at dp <= 64 in LDS, above in the wave's own rows of its partial slot.
constexpr bool half_sums_in_lds(int kb) { return kb <= 4; }

template <int KB, int TAIL, int NI, int WAVES, int NB, bool AHEAD, int MINW, int KIND, bool FAR>
__global__ __launch_bounds__(WAVES * kWave, MINW) void pair_half_kernel(
    const float* __restrict__ ps, const float* __restrict__ pn, const float* __restrict__ xs, const float* __restrict__ xt,
    const float* __restrict__ xn, float* __restrict__ part_t, float* __restrict__ part_d,
    int ntiles, int tiles_per_split, int nsplit, int64_t m_pad, float laplace_c0, float* __restrict__ part_shift)
{
    static_assert(NI % 2 == 0 && NI % NB == 0, "a wave's own rows are whole chunks");
    static_assert((KB % 2 != 0) == (TAIL == kTailSixteen || TAIL == kTailEight), "an odd block count has a tail");
    constexpr bool SCORE = KIND == kScoreSelf || KIND == kScorePoints;
    constexpr bool SELF = KIND == kScoreSelf;
    constexpr bool LAPLACE = KIND == kEvalLaplace;
    static_assert(KIND != kRowMax, "shifted sums find their shifts as they go");
    constexpr bool ODD = HalfRows<KB, TAIL, NI, SCORE, FAR>::ODD, TERMED = TAIL != kTailNone;
    constexpr int DP = KB * 16;
    constexpr int KT = SCORE ? KB : 1;
    constexpr int PAIRS = KB / 2;
    constexpr int XCH = 2 * KB + (ODD ? 1 : 0), TCH = 3 * KB;    // 1 KiB pieces of a chunk of xs (the tail's last one: half), of xt
    constexpr int CH = SCORE ? XCH + TCH : XCH;
    constexpr int STAGE = (CH + WAVES - 1) / WAVES;              // pieces a wave moves per chunk
    constexpr bool SUMLDS = SCORE && half_sums_in_lds(KB);
    __shared__ __align__(16) char stage_lds[2][CH * kPartBytes];
    __shared__ f32x4 sum_lds[SUMLDS ? WAVES : 1][SUMLDS ? NI * KT : 1][SUMLDS ? kWave : 1];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);    // wave-uniform by construction
    const int r = lane & 15, g = lane >> 4;
    const int split = blockIdx.x % nsplit;
    const int64_t row_block = blockIdx.x / nsplit;
    const int64_t row0 = (row_block * WAVES + wave) * (NI * kTile);

    const int c_begin = split * tiles_per_split / 2;
    const int c_end = min(ntiles, split * tiles_per_split + tiles_per_split) / 2;
    uint32_t marks = 0;                                     // of the split's samples (wave-uniform), where they are asked for
    const int64_t n_pad = ((int64_t)ntiles * kTile + kRowPad - 1) / kRowPad * kRowPad;
    const uint8_t* const marks_at = half2_marks(const_cast<float*>(xs), n_pad, DP);
    const float* const units = half2_units(const_cast<float*>(xs), n_pad, DP);
    const float other_units = SCORE ? units[DP] : 0.0f;             // a column of xt is not in plain coordinates

    HalfRows<KB, TAIL, NI, SCORE, FAR> rows;
    rows.load(ps, pn, row0, r, g);
    // FAR: a row may be held as 2^-k times itself, 2^k behind the prepared rows, and so may samples; far: one of the wave's rows
    // is, or no sample that its first look has seen is within kFarShift of one, and exponents are shifted last (wave-uniform).
    // (Without such a row samples that are held so have no weight.)
    bool far = false;
    const float* const pscale = FAR ? half2_scale(const_cast<float*>(ps), m_pad, DP) : nullptr;
    const float* const xscale = FAR ? half2_scale(const_cast<float*>(xs), n_pad, DP) : nullptr;
    auto of_row = [&](const float* at, int t) { return load_at<float>(reinterpret_cast<const char*>(at + row0 + t * kTile), r * 4u); };
    if constexpr (FAR) {
#pragma unroll
        for (int t = 0; t < NI; ++t) far |= __builtin_amdgcn_ballot_w64(of_row(pscale, t) != 1.0f) != 0;
        if (SCORE && far) rows.bare(g);
    }

    // Two-level accumulation: the running sums (tacc, dacc) are folded into a second level every kFlushTiles sample
    // tiles, so no fp32 accumulator sees more than a short chain of additions at its own magnitude.
    f32x4 tacc[NI][KT];
    float dacc[NI], dsum[NI];
    float lc0[LAPLACE ? NI : 1];          // Laplace factor constant per row tile: 1 + d/2 + shift_i ln 2
    float unit[SCORE ? NI : 1];           // what a W of one is worth
    float less[FAR ? NI : 1];             // FAR: by how much the exponents have been lowered, the rows' shift
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        dacc[t] = dsum[t] = 0.0f;
#pragma unroll
        for (int mb = 0; mb < KT; ++mb) {
            tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (SUMLDS) sum_lds[wave][t * KT + mb][lane] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (LAPLACE) {
            lc0[t] = laplace_c0;
            asm("" : "+v"(lc0[t]));        // in a register a row tile: as one scalar for all the compiler schedules the loop 2 % worse
        }
        if (SCORE) unit[t] = kWeightScale;
        if (FAR) less[t] = 0.0f;
    }
    auto slot_at = [&](int t, int mb) {
        return reinterpret_cast<f32x4*>(part_t + ((int64_t)split * m_pad + row0 + t * kTile + r) * DP + g * 4 + mb * 16);
    };
    // the lane's offsets into a sample tile's operands of the tail
    const int tail_first = PAIRS * 2048 + lane * 16;
    const int tail_term = PAIRS * 2048 + r * 16 + (TAIL == kTailSixteen ? (g < 2 ? g * 256 : g == 2 ? 1024 : 512) : (g < 2 ? 0 : g == 2 ? 512 : 1024));

    constexpr int GROUPS = PAIRS + (ODD ? 1 : 0);
    constexpr int STEPS = 2 * GROUPS - 1;      // leading products of all groups but the last, the last, the others' rest
    // Operands of one group of MFMAs; scheduling barriers keep an early read early.
    f16x8 ga[2][2][2], ta[2][3];
    auto pin = [] { if (AHEAD) __builtin_amdgcn_sched_barrier(0); };
    auto read_gram = [&](const char* xc, int s, f16x8 (&a)[2][2]) __attribute__((always_inline)) {
        if (GROUPS == 2 && s == GROUPS) return;             // still there from the first step
        const int p = s < GROUPS ? s : s - GROUPS;
        const int parts = GROUPS > 2 && s < GROUPS - 1 ? 1 : 2;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const char* base = xc + u * half_tile_bytes(KB);
            if (p < PAIRS) {
#pragma unroll
                for (int q = 0; q < parts; ++q) a[u][q] = *reinterpret_cast<const f16x8*>(base + p * 2048 + q * 1024 + lane * 16);
            } else {
                if (TAIL == kTailSixteen) a[u][0] = *reinterpret_cast<const f16x8*>(base + tail_first);
                a[u][1] = *reinterpret_cast<const f16x8*>(base + tail_term);
            }
        }
    };
    auto read_t = [&](const char* xc, int mb, f16x8 (&a)[3]) {
#pragma unroll
        for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const f16x8*>(xc + XCH * kPartBytes + mb * 3072 + q * kPartBytes + lane * 16);
    };
    // SCORE: the power of two by which a row's exponents are lowered (kept as what a w of one is worth)
    auto lowered = [&](int t) { return (float)((int)(__builtin_bit_cast(uint32_t, unit[SCORE ? t : 0]) >> 23) - 127 - 11); };
    // Exponents of NB row tiles from t0 on against a chunk's two sample tiles.  own (SELF): the row tile that is the chunk's
    // first sample tile, if it is one.  c_at: the chunk.  to_t: the first operands of the second contraction are read behind.
    auto exponents = [&](const char* xc, int c_at, int t0, const f32x4& nj0, const f32x4& nj1, int own, bool to_t, f32x4 (&c)[NB][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            const float add = TERMED ? 0.0f : rows.term[t0 + t];
            c[t][0] = FAR && far ? f32x4{0.f, 0.f, 0.f, 0.f} : TERMED ? nj0 : nj0 + add;
            c[t][1] = FAR && far ? f32x4{0.f, 0.f, 0.f, 0.f} : TERMED ? nj1 : nj1 + add;
        }
        if (AHEAD) read_gram(xc, 0, ga[0]);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (!AHEAD) read_gram(xc, s, ga[s & 1]);
            else if (s + 1 < STEPS) read_gram(xc, s + 1, ga[(s + 1) & 1]);
            else if (to_t) read_t(xc, 0, ta[0]);
            pin();
            const f16x8 (&a)[2][2] = ga[s & 1];
            // the largest products of all groups and the row's term first: they bring the accumulator from the size
            // of the norms down to that of the distance, where the small ones round finer
            const int p = s < GROUPS ? s : s - GROUPS;
            const int k0 = s < GROUPS ? 0 : 1, k1 = s < GROUPS - 1 ? 1 : 3;
            if (p < PAIRS) {
                constexpr int PA[3] = {0, 1, 0}, PB[3] = {0, 0, 1};
#pragma unroll
                for (int k = k0; k < k1; ++k)
#pragma unroll
                    for (int t = 0; t < NB; ++t)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            c[t][u] = mfma_f16(a[u][PA[k]], rows.b[t0 + t][p < PAIRS ? p : 0][PB[k]], c[t][u]);
            } else {
#pragma unroll
                for (int k = TAIL == kTailSixteen ? 0 : 1; k < 2; ++k)
#pragma unroll
                    for (int t = 0; t < NB; ++t)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            c[t][u] = mfma_f16(a[u][k], rows.o[ODD ? t0 + t : 0][TAIL == kTailSixteen ? k : 0], c[t][u]);
            }
            pin();
        }
        if (FAR && __builtin_expect(far, 0)) {
            // such rows' exponents are rounded at the size of the norms, the same way whatever the shift, and only then shifted:
            // with the shift in the row's term a look for the largest and the weights would miss each other
            // (samples that are held as they are have a scale of 1)
            f32x4 xs[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) xs[u] = load_at<f32x4>(reinterpret_cast<const char*>(xscale + (int64_t)c_at * kChunkRows + u * kTile), g * 16u);
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const float unscale = of_row(pscale, t0 + t), base = of_row(pn, t0 + t);
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    const float norm = v < 4 ? nj0[v % 4] : nj1[v % 4];
                    c[t][v / 4][v % 4] = (fmaf(c[t][v / 4][v % 4], unscale * xs[v / 4][v % 4], norm) + base) - less[FAR ? t0 + t : 0];
                }
            }
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
    };
    // a row's largest exponent of a chunk (largest of the lane's eight: its share of the row)
    auto largest = [&](const f32x4 (&c)[2]) {
        float most = c[0][0];
#pragma unroll
        for (int v = 1; v < 8; ++v) most = fmaxf(most, c[v / 4][v % 4]);
        most = fmaxf(most, __shfl_xor(most, 16));
        return fmaxf(most, __shfl_xor(most, 32));
    };
    // SCORE: by how much a row's exponents have to be lowered
    auto excess = [&](const f32x4 (&c)[2]) { return floorf(largest(c)) - (float)kRaisedTo; };
    // SCORE: sets row tile t's scale: exponents are 2^-low of what they stand for.  The term anew from the norm: sums of it with
    // several shifts, one after the other, would round every time (2^-18 with a norm of 30 and the shift of 126 that suits any
    // point: score errors of up to 2.4 times the present ones).
    auto set_scale = [&](int t, float low, float norm, float residual) {
        rows.term[t] = norm - low;
        unit[SCORE ? t : 0] = ldexpf(kWeightScale, (int)low);
        rows.place_term(t, rows.term[t], residual, g);
    };
    // FAR: the same with a shift of any size, which the sums are kept relative to and which goes with them to the slots.  What
    // rounding norm - low leaves goes into the term's third part; without a term in columns (shift_rest) the sums make up for it.
    auto shift_rest = [&](float norm, float low) {
        const float term = norm - low, back = term - norm, rest = (norm - (term - back)) + (-low - back);
        return fabsf(rest) < 500.0f ? rest : 0.0f;          // (more: there is no sample yet that the shift could be of)
    };
    auto set_shift = [&](int t, float low) {
        const int64_t row = row0 + t * kTile + r;
        const float norm = pn[row];
        less[FAR ? t : 0] = low;
        rows.term[t] = norm - low;
        if (LAPLACE) lc0[LAPLACE ? t : 0] = fmaf(low, kLn2, laplace_c0);
        if (TERMED) rows.place_term(t, far ? 0.0f : rows.term[t], far ? 0.0f : shift_rest(norm, low) + (SCORE ? rows.residual(ps, row) : 0.0f), g);
    };
    // (above 2^24, where floats are further apart than kRaisedTo, a difference could come out that much too low)
    auto shift_for = [&](float most) {
        const float put = SCORE ? (float)kRaisedTo : 0.0f, low = floorf(most) - put;
        return most - low <= put + 1.0f ? low : floorf(most);
    };
    auto rest_of = [&](int t) { return TERMED || far ? 0.0f : shift_rest(of_row(pn, t), less[FAR ? t : 0]); };

    bool flushed = false;                                   // !SUMLDS: the partial slot holds second-level sums
    // One chunk against all NI row tiles.
    auto chunk = [&](const char* xc, int c_at, const f32x4& nj0, const f32x4& nj1, int own) __attribute__((always_inline)) {
#pragma unroll
        for (int t0 = 0; t0 < NI; t0 += NB) {
            f32x4 c[NB][2], phi[NB][2];
            float dt[NB];
            exponents(xc, c_at, t0, nj0, nj1, own, SCORE, c);
            auto weigh = [&](int t) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) phi[t][u][v] = __builtin_amdgcn_exp2f(c[t][u][v]);
                if (LAPLACE) {
                    // c is the base-2 exponent -r^2/(2h^2) log2(e) (less the row's shift), so the Laplace factor
                    // 1 + d/2 - r^2/(2h^2) is lc0 + c ln 2 (Laplace-corrected KDE section)
                    if (FAR) dt[t] = 0.0f;
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        const float factor = fmaf(c[t][v / 4][v % 4], kLn2, lc0[LAPLACE ? t0 + t : 0]);
                        if constexpr (FAR) dt[t] = fmaf(phi[t][v / 4][v % 4], factor, dt[t]);
                        else dacc[t0 + t] = fmaf(phi[t][v / 4][v % 4], factor, dacc[t0 + t]);
                    }
                } else {
                    dt[t] = ((phi[t][0].x + phi[t][0].y) + (phi[t][0].z + phi[t][0].w)) +
                            ((phi[t][1].x + phi[t][1].y) + (phi[t][1].z + phi[t][1].w));
                }
            };
            [[maybe_unused]] float all = 0.0f;
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                weigh(t);
                // SCORE: the largest of the rows that a lane holds: fmaxf passes a NaN over, beside which a sum would see no other row.
                // (Without Phi X what leaves the range, and NaN, has to be seen; a signed sum near zero does no harm.)
                if (SCORE) all = t == 0 ? dt[t] : fmaxf(all, dt[t]);
                else if (FAR) all = t == 0 ? (LAPLACE ? fabsf(dt[t]) : dt[t]) : all + (LAPLACE ? fabsf(dt[t]) : dt[t]);
            }
            // a weight may have outgrown its row's scale: that row's exponents are lowered, its largest W is 2^kRaisedTo
            // again (wave-uniform; in place, so that nothing is copied where it does not happen)
            if (SCORE && !FAR && __builtin_expect(__builtin_amdgcn_ballot_w64(all > kMostWeight) != 0, 0)) {
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    const float up = fminf(fmaxf(excess(c[t]), 0.0f), 16384.0f);
                    const int64_t row = row0 + (t0 + t) * kTile + r;
                    set_scale(t0 + t, lowered(t0 + t) + up, pn[row], rows.residual(ps, row));
#pragma unroll
                    for (int u = 0; u < 2; ++u) c[t][u] -= up;
                    weigh(t);
                }
            }
            // FAR: or the shift may; what has been summed, on both levels, is brought to the new one.  A shift too large, or a
            // weight too far out, for the difference to be exact: the row is looked at anew.
            if (FAR && __builtin_expect(__builtin_amdgcn_ballot_w64(SCORE ? all > kMostWeight : !(all <= kMostShifted)) != 0, 0)) {
                float before[NB], by[NB], up[NB];
                bool exact = true;
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    before[t] = less[FAR ? t0 + t : 0];
                    by[t] = rest_of(t0 + t);
                    up[t] = fmaxf(floorf(largest(c[t])) - (SCORE ? (float)kRaisedTo : 0.0f), 0.0f);
                    exact &= up[t] < 16384.0f && fabsf(before[t]) < 4194304.0f;
                }
                exact = __builtin_amdgcn_ballot_w64(!exact) == 0;
                if (!exact) {
#pragma unroll
                    for (int t = 0; t < NB; ++t) set_shift(t0 + t, 0.0f);
                    exponents(xc, c_at, t0, nj0, nj1, own, false, c);
                }
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    set_shift(t0 + t, exact ? before[t] + up[t] : fmaxf(before[t], shift_for(largest(c[t]))));
                    const float now = less[FAR ? t0 + t : 0];
                    by[t] = __builtin_amdgcn_exp2f((before[t] - now) + (by[t] - rest_of(t0 + t)));
#pragma unroll
                    for (int u = 0; u < 2; ++u) c[t][u] -= exact ? up[t] : 0.0f;
                    dacc[t0 + t] *= by[t];
                    dsum[t0 + t] *= by[t];
                    if constexpr (SCORE) {
#pragma unroll
                        for (int mb = 0; mb < KT; ++mb) {
                            tacc[t0 + t][mb] *= by[t];
                            if (SUMLDS) sum_lds[wave][(t0 + t) * KT + mb][lane] *= by[t];
                            else if (flushed) *slot_at(t0 + t, mb) *= by[t];
                        }
                    }
                }
                if (!exact) exponents(xc, c_at, t0, nj0, nj1, own, false, c);
                if (SCORE && AHEAD) read_t(xc, 0, ta[0]);       // (their registers are not kept for this rare path)
#pragma unroll
                for (int t = 0; t < NB; ++t) weigh(t);
            }
            if constexpr (SCORE) {
                f16x8 w[NB][2];
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    dacc[t0 + t] = FAR ? dacc[t0 + t] + dt[t] : fmaf(dt[t], unit[t0 + t], dacc[t0 + t]);      // kWeightScale times D
                    // keeps the sum here: the compiler would otherwise sink it behind the MFMAs and hold the Phi tiles live
                    asm volatile("" : "+v"(dacc[t0 + t]));
                    split_weights(phi[t][0], phi[t][1], w[t][0], w[t][1]);
                }
                f32x4 sum[2][NB];
                auto add = [&](int mb) {
#pragma unroll
                    for (int t = 0; t < NB; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            tacc[t0 + t][mb][v] = FAR ? sum[mb & 1][t][v] + tacc[t0 + t][mb][v] : fmaf(sum[mb & 1][t][v], unit[t0 + t], tacc[t0 + t][mb][v]);
                };
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) {
                    if (!AHEAD) read_t(xc, mb, ta[mb & 1]);
                    else if (mb + 1 < KB) read_t(xc, mb + 1, ta[(mb + 1) & 1]);
                    pin();
                    const f16x8 (&a)[3] = ta[mb & 1];
                    // The chunk's sum starts from zero, its smallest products first: an MFMA rounds its accumulator after
                    // every lane group (four times), which this way happens at the size of 32 terms and not of the
                    // running sum.
                    constexpr int PA[3] = {2, 1, 0}, PB[3] = {1, 0, 0};
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int t = 0; t < NB; ++t)
                            sum[mb & 1][t] = mfma_f16(a[PA[k]], w[t][PB[k]], k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[mb & 1][t]);
                    pin();
                    // added a group later, when the MFMAs have finished
                    if (mb > 0) add(mb - 1);
                }
                add(KB - 1);
            } else if constexpr (!LAPLACE || FAR) {
#pragma unroll
                for (int t = 0; t < NB; ++t) dacc[t0 + t] += dt[t];
            }
        }
    };

    const int own0 = (int)(row0 / kChunkRows);              // SELF: the wave's own rows are chunks own0 .. own0 + NI/2 - 1
    const char* const xs_b = reinterpret_cast<const char*>(xs);
    const char* const xt_b = reinterpret_cast<const char*>(xt);
    if (c_begin < c_end) {
        const int c_last = c_end - 1;                       // the prefetch past the end re-reads the last chunk (in bounds)
        // The pieces a wave moves: one scalar base and stride each (no branches in the loop).  A piece past the end is the
        // last one again, deposited twice with the same bytes.
        auto piece_of = [&](int q) { return (q + 1) * WAVES <= CH ? q * WAVES + wave : min(q * WAVES + wave, CH - 1); };
        const uint32_t lane16 = lane * 16u;
        f32x4 stage[STAGE];
        auto fetch = [&](int c) {
            const char* const at_x = xs_b + (int64_t)min(c, c_last) * (2 * half_tile_bytes(KB));
            const char* const at_t = xt_b + (int64_t)min(c, c_last) * (TCH * kPartBytes);
#pragma unroll
            for (int q = 0; q < STAGE; ++q) {
                const int piece = piece_of(q);                              // wave-uniform
                stage[q] = load_at<f32x4>(SCORE && piece >= XCH ? at_t + (piece - XCH) * kPartBytes : at_x + piece * kPartBytes, lane16);
            }
        };
        auto deposit = [&](char* buf) {
#pragma unroll
            for (int q = 0; q < STAGE; ++q) *reinterpret_cast<f32x4*>(buf + piece_of(q) * kPartBytes + lane16) = stage[q];
        };
        auto norms = [&](int c, int u) {
            return load_at<f32x4>(reinterpret_cast<const char*>(xn + (int64_t)min(c, c_last) * kChunkRows), u * kTile * 4 + g * 16u);
        };
        f32x4 nj0 = norms(c_begin, 0), nj1 = norms(c_begin, 1);
        fetch(c_begin);                                     // (all first loads are under way before the first is waited for)
        float residual[SCORE && !FAR ? NI : 1];
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            if (SCORE && !FAR) residual[SCORE && !FAR ? t : 0] = rows.residual(ps, row0 + t * kTile + r);
            rows.place_term(t, FAR && far ? 0.0f : rows.term[t], 0.0f, g);
        }
        if (FAR) marks = marks_of(marks_at, c_begin, c_end, lane);
        deposit(stage_lds[0]);
        __syncthreads();
        if constexpr (SCORE && !FAR) {
            // every row's scale, from its largest weight among the first chunk's samples (without a near one: the smallest)
#pragma unroll
            for (int t0 = 0; t0 < NI; t0 += NB) {
                f32x4 c[NB][2];
                exponents(stage_lds[0], c_begin, t0, nj0, nj1, 2 * (c_begin - own0), false, c);
#pragma unroll
                for (int t = 0; t < NB; ++t)
                    set_scale(t0 + t, fminf(fmaxf(excess(c[t]), kLeastShift), 16384.0f), rows.term[t0 + t], residual[SCORE && !FAR ? t0 + t : 0]);
            }
        }
        if constexpr (FAR) {
            // every row's shift, from its largest exponent among the first chunk's samples; where that is below kFarShift, once more
            // with the exponents of far rows
            auto look = [&] {
                bool below = false;
#pragma unroll
                for (int t0 = 0; t0 < NI; t0 += NB) {
                    f32x4 c[NB][2];
                    exponents(stage_lds[0], c_begin, t0, nj0, nj1, 0, false, c);
#pragma unroll
                    for (int t = 0; t < NB; ++t) {
                        const float most = largest(c[t]);
                        // (a padding row is far from everything, and nothing for its neighbours in the wave to follow; its term is still its norm here)
                        below |= __builtin_amdgcn_ballot_w64(most < kFarShift && rows.term[t0 + t] != kPadNorm) != 0;
                        set_shift(t0 + t, fmaxf(shift_for(most), kNegHuge));
                    }
                }
                return below;
            };
            if (look() && !far && (marks & kMarkDistant) != 0) {
                far = true;
                if (SCORE) rows.bare(g);
#pragma unroll
                for (int t = 0; t < NI; ++t) set_shift(t, 0.0f);
                look();
            }
        }
        // SCORE: a chunk with units of its own is summed in them: what has been summed is brought to them and back, on both levels.
        // Where the split has one every chunk is a turn of the outer loop.  (Asked inside the inner one it cost 3 to 5 % of a score.)
        auto own_units = [&](int c, bool to) __attribute__((always_inline)) {
            if (!(marks & marks_at[2 * c] & kMarkOwnUnits)) return;
#pragma unroll
            for (int mb = 0; mb < KT; ++mb) {
                f32x4 by = load_at<f32x4>(reinterpret_cast<const char*>(units + 2 * DP + 4 + (int64_t)c * DP + mb * 16), g * 16u);
                if (to) by = f32x4{inverse_unit(by.x), inverse_unit(by.y), inverse_unit(by.z), inverse_unit(by.w)};
#pragma unroll
                for (int t = 0; t < NI; ++t) {
                    tacc[t][mb] *= by;
                    if (SUMLDS) sum_lds[wave][t * KT + mb][lane] *= by;
                    else if (flushed) *slot_at(t, mb) *= by;
                }
            }
        };
        if (SCORE && !FAR && other_units != 0.0f) marks = marks_of(marks_at, c_begin, c_end, lane);
        const bool alone = SCORE && (marks & kMarkOwnUnits) != 0;
        for (int c = c_begin; c < c_end;) {
            const int end = alone ? c + 1 : c_end;
            if (SCORE && alone) own_units(c, true);
            for (; c < end; ++c) {                          // the same bounds for all waves of the workgroup
                const char* cur = stage_lds[(c - c_begin) & 1];
                fetch(c + 1);                               // lands in registers while this chunk is worked on
                const f32x4 nn0 = norms(c + 1, 0), nn1 = norms(c + 1, 1);
                chunk(cur, c, nj0, nj1, 2 * (c - own0));
                if (((c + 1 - c_begin) & (kFlushTiles / 2 - 1)) == 0) {
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
            if (SCORE && alone) own_units(end - 1, false);
        }
    }
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        const float by = FAR ? __builtin_amdgcn_exp2f(rest_of(t)) : 1.0f;
        if constexpr (SCORE) {
#pragma unroll
            for (int mb = 0; mb < KT; ++mb) {
                if (SUMLDS) tacc[t][mb] += sum_lds[wave][t * KT + mb][lane];
                else if (flushed) tacc[t][mb] += *slot_at(t, mb);
                if (FAR) tacc[t][mb] *= by;
                *slot_at(t, mb) = tacc[t][mb];
            }
        }
        // D needs the sum over the four lane groups g
        float dtot = (dsum[t] + dacc[t]) * (SCORE ? 1.0f / kWeightScale : 1.0f);
        if (FAR) dtot *= by;
#pragma unroll
        for (int step = 16; step <= 32; step *= 2) dtot += __shfl_xor(dtot, step);
        if (SCORE && other_units != 0.0f) dtot = -dtot;         // tells the epilogues
        if (g == 0) {
            const int64_t at = (int64_t)split * m_pad + row0 + t * kTile + r;
            part_d[at] = dtot;
            if (FAR) part_shift[at] = c_begin < c_end ? less[FAR ? t : 0] : kNegHuge;
        }
    }
}

}  // namespace
