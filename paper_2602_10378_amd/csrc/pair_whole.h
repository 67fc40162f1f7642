// Pair kernel of the fp32 matrix path for small sample sets: a workgroup sums a few rows over all samples and writes the outputs.
//
// What bounds a small call is its chain of dependent launches, 4 to 6 us each (preparation, pairs, reduction of the split slots, and
// for the one-call pass the same again), beside pair work of 1 to 10 us.  Here the waves of a workgroup share its rows and divide the
// samples, chunk by chunk, among themselves; their sums meet in LDS, and the workgroup goes on to the outputs: no split slots, no
// launch for their reduction, and in the one-call pass none for the preparation of the shifted samples either (FIT).  A call is two
// launches, sdkde_fit_eval three.  Every wave has samples of its own, so operands go from the caches straight to registers, and a
// row tile a wave is what fills the chip with few rows; the price, operand reads that nothing amortises, is why larger sets keep
// the kernels of pair_half.h (whole_row_tiles in sdkde.hip says where the line is, with both sides measured).
// The arithmetic of a chunk is that of pair_half_kernel: order of the part products, scale of the weights, units of narrow columns.
#pragma once
#include "common.h"
#include "epilogue.h"
#include "half2.h"
#include "pair_half.h"
#include "prep.h"

namespace {

// Where the results go and what they are formed with.
struct WholeOut {
    int d;
    float min_sum;                         // least_trusted_sum of the sample count
    // scores
    float inv_ah2, half_h2;
    float* score;                          // optional
    const float* x;                        // the samples themselves, for
    float* x_sd;                           // the shifted ones (optional, at the samples only)
    int quad_io;                           // d is a multiple of four and these arrays are 16-byte aligned
    ScoreUnits units;
    // densities
    double lognorm;
    const float* residual;
    float *density, *log_density;          // optional, one at least
    // FIT: the preparation of the shifted samples
    PrepJob sd_job;
    const float* centre;
    double a;
    Stamp stamp;
};

// Waves of a workgroup: as many as have the registers that a chunk's operands take.
constexpr int whole_waves(int kb, int row_tiles) { return kb <= 2 && row_tiles == 1 ? 16 : 8; }
// Most chunks a wave sums in one level (the larger kernels fold their sums as often, kFlushTiles).
constexpr int kWholeChunks = kFlushTiles / 2;

template <int KB, int TAIL, int NI, int KIND, bool FIT>
__global__ __launch_bounds__(whole_waves(KB, NI) * kWave) void pair_whole_kernel(
    const float* __restrict__ ps, const float* __restrict__ pn, const float* __restrict__ xs, const float* __restrict__ xt,
    const float* __restrict__ xn, int nchunks, int64_t n_pad, int64_t m, int64_t m_pad, float laplace_c0, WholeOut out)
{
    static_assert((KB % 2 != 0) == (TAIL == kTailSixteen || TAIL == kTailEight), "an odd block count has a tail");
    static_assert(!FIT || (KIND == kScoreSelf && NI == 1), "shifted samples are those of the score at the samples, a tile a workgroup");
    constexpr int WAVES = whole_waves(KB, NI), THREADS = WAVES * kWave;
    constexpr bool SCORE = KIND == kScoreSelf || KIND == kScorePoints;
    constexpr bool SELF = KIND == kScoreSelf, LAPLACE = KIND == kEvalLaplace;
    using Rows = HalfRows<KB, TAIL, NI, SCORE, false>;
    constexpr bool ODD = Rows::ODD, TERMED = TAIL != kTailNone;
    constexpr int DP = KB * 16, PAIRS = KB / 2, KT = SCORE ? KB : 1;
    constexpr int TAIL_OPS = TAIL == kTailSixteen ? 2 : ODD ? 1 : 0, OPS = 2 * PAIRS + TAIL_OPS;     // operands of a sample tile
    constexpr int DEPTH = KB <= 4 ? (SCORE ? 2 : 3) : 1;        // chunks whose operands are in registers or on the way
    constexpr bool HALVE = KB > 4;                  // sums of two waves are added before all meet in LDS
    constexpr int SLOTS = HALVE ? WAVES / 2 : WAVES;
    constexpr int ITEMS = NI * KT * kWave;          // four columns of a row each
    static_assert(ITEMS <= THREADS && NI * kTile <= THREADS, "an output a thread");
    __shared__ f32x4 sum_t[SCORE ? SLOTS : 1][SCORE ? NI * KT : 1][SCORE ? kWave : 1];
    __shared__ float sum_d[WAVES][NI * kTile];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r = lane & 15, g = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.x * (NI * kTile);
    const uint32_t lane16 = lane * 16u;
    const char* const xs_b = reinterpret_cast<const char*>(xs);
    const char* const xt_b = reinterpret_cast<const char*>(xt);

    struct Operands {
        f16x8 a[2][OPS];
        f32x4 nj[2];
        f16x8 x[KT][2];
    };
    const uint32_t tail_first = PAIRS * 2048 + lane16;
    const uint32_t tail_term = PAIRS * 2048 + r * 16u + (TAIL == kTailSixteen ? (g < 2 ? g * 256u : g == 2 ? 1024u : 512u) : (g < 2 ? 0u : g == 2 ? 512u : 1024u));
    auto read = [&](int c, Operands& o) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const char* const base = xs_b + ((int64_t)c * 2 + u) * half_tile_bytes(KB);
#pragma unroll
            for (int k = 0; k < 2 * PAIRS; ++k) o.a[u][k] = load_at<f16x8>(base, k * 1024u + lane16);
            if (TAIL == kTailSixteen) o.a[u][2 * PAIRS] = load_at<f16x8>(base, tail_first);
            if (ODD) o.a[u][OPS - 1] = load_at<f16x8>(base, tail_term);
            o.nj[u] = load_at<f32x4>(reinterpret_cast<const char*>(xn + (int64_t)c * kChunkRows), u * kTile * 4 + g * 16u);
        }
        if constexpr (SCORE) {
            const char* const base = xt_b + (int64_t)c * (KB * 3072);
#pragma unroll
            for (int mb = 0; mb < KB; ++mb)
#pragma unroll
                for (int q = 0; q < 2; ++q) o.x[mb][q] = load_at<f16x8>(base, mb * 3072u + q * 1024u + lane16);
        }
    };

    // FIT covers the padding rows, too, which have no sums
    // A wave's chunks are wave, wave + WAVES, ..., and workgroups of one XCD (every eighth) start at different ones of them, so that
    // their first reads together bring all samples into its cache: left there by a launch on all XCDs, they are a miss to each.
    const int steps = row0 < m && wave < nchunks ? (nchunks - wave - 1) / WAVES + 1 : 0, turn = steps ? blockIdx.x / 8 % steps : 0;
    auto chunk_at = [&](int step) { return wave + (step + turn < steps ? step + turn : step + turn - steps) * WAVES; };
    Operands ring[DEPTH];
    if (steps > 0) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) read(chunk_at(min(k, steps - 1)), ring[k]);
    }
    Rows rows;
    rows.load(ps, pn, row0, r, g);
    float norm[NI], residual[NI], unit[NI], dacc[NI];
    f32x4 tacc[NI][KT];
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        norm[t] = rows.term[t];
        residual[t] = SCORE ? rows.residual(ps, row0 + t * kTile + r) : 0.0f;
        rows.place_term(t, norm[t], residual[t], g);
        unit[t] = kWeightScale;
        dacc[t] = 0.0f;
#pragma unroll
        for (int mb = 0; mb < KT; ++mb) tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float* const units = half2_units(const_cast<float*>(xs), n_pad, DP);
    const uint8_t* const marks_at = half2_marks(const_cast<float*>(xs), n_pad, DP);
    const float other_units = SCORE ? units[DP] : 0.0f;
    const bool alone = SCORE && other_units != 0.0f && (marks_of(marks_at, 0, nchunks, lane) & kMarkOwnUnits) != 0;
    const int tile0 = (int)(row0 / kTile);

    auto chunk = [&](int c, bool first, const Operands& now) __attribute__((always_inline)) {
        f32x4 e[NI][2];                             // exponents
        auto exponents = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NI; ++t)
#pragma unroll
                for (int u = 0; u < 2; ++u) e[t][u] = TERMED ? now.nj[u] : now.nj[u] + rows.term[t];
            auto product = [&](int p, int k) __attribute__((always_inline)) {       // of 32-column block p: h h, l h, h l
                constexpr int PA[3] = {0, 1, 0}, PB[3] = {0, 0, 1};
#pragma unroll
                for (int t = 0; t < NI; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u) e[t][u] = mfma_f16(now.a[u][2 * p + PA[k]], rows.b[t][p][PB[k]], e[t][u]);
            };
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) product(p, 0);
            if constexpr (ODD) {
#pragma unroll
                for (int k = 0; k < TAIL_OPS; ++k)
#pragma unroll
                    for (int t = 0; t < NI; ++t)
#pragma unroll
                        for (int u = 0; u < 2; ++u) e[t][u] = mfma_f16(now.a[u][2 * PAIRS + k], rows.o[t][k], e[t][u]);
            }
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                product(p, 1);
                product(p, 2);
            }
            const int own = 2 * c - tile0;              // the row tile that is the chunk's first sample tile (wave-uniform)
            if (SELF && own > -2 && own < NI) {
#pragma unroll
                for (int t = 0; t < NI; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (own + u == t) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) e[t][u][v] = g * 4 + v == r ? kNegHuge : e[t][u][v];
                        }
            }
        };
        exponents();
        f32x4 phi[NI][2];
        float dt[NI];
        auto weigh = [&](int t) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < 8; ++v) phi[t][v / 4][v % 4] = __builtin_amdgcn_exp2f(e[t][v / 4][v % 4]);
            if (LAPLACE) {
                dt[t] = 0.0f;
#pragma unroll
                for (int v = 0; v < 8; ++v) dt[t] = fmaf(phi[t][v / 4][v % 4], fmaf(e[t][v / 4][v % 4], kLn2, laplace_c0), dt[t]);
            } else {
                dt[t] = ((phi[t][0].x + phi[t][0].y) + (phi[t][0].z + phi[t][0].w)) + ((phi[t][1].x + phi[t][1].y) + (phi[t][1].z + phi[t][1].w));
            }
        };
        // SCORE: the scale of a row's weights, see pair_half.h: set from the first chunk's largest, raised when a weight outgrows it
        auto lower = [&](float least) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NI; ++t) {
                float most = e[t][0][0];
#pragma unroll
                for (int v = 1; v < 8; ++v) most = fmaxf(most, e[t][v / 4][v % 4]);
                most = fmaxf(most, __shfl_xor(most, 16));
                most = fmaxf(most, __shfl_xor(most, 32));
                const float up = fminf(fmaxf(floorf(most) - (float)kRaisedTo, least), 16384.0f);
                const float low = (float)((int)(__builtin_bit_cast(uint32_t, unit[t]) >> 23) - 127 - 11) + up;
                rows.term[t] = norm[t] - low;
                unit[t] = ldexpf(kWeightScale, (int)low);
                rows.place_term(t, rows.term[t], residual[t], g);
#pragma unroll
                for (int u = 0; u < 2; ++u) e[t][u] -= up;
            }
        };
        if (SCORE && first) {
            lower(kLeastShift);
            exponents();            // beside a term as large as the norms an MFMA truncates the small products (score errors 1.02 to 1.05 times as large)
        }
        [[maybe_unused]] float all = 0.0f;
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            weigh(t);
            all = t == 0 ? dt[t] : fmaxf(all, dt[t]);          // (not a sum: see pair_half.h)
        }
        if (SCORE && __builtin_expect(__builtin_amdgcn_ballot_w64(all > kMostWeight) != 0, 0)) {
            lower(0.0f);
#pragma unroll
            for (int t = 0; t < NI; ++t) weigh(t);
        }
        if constexpr (SCORE) {
            f32x4 by[KT];
            const bool own_units = alone && (marks_at[2 * c] & kMarkOwnUnits) != 0;         // of this chunk (wave-uniform)
            if (__builtin_expect(own_units, 0)) {
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) {
                    by[mb] = load_at<f32x4>(reinterpret_cast<const char*>(units + 2 * DP + 4 + (int64_t)c * DP + mb * 16), g * 16u);
#pragma unroll
                    for (int t = 0; t < NI; ++t)
                        tacc[t][mb] *= f32x4{inverse_unit(by[mb].x), inverse_unit(by[mb].y), inverse_unit(by[mb].z), inverse_unit(by[mb].w)};
                }
            }
#pragma unroll
            for (int t = 0; t < NI; ++t) {
                dacc[t] = fmaf(dt[t], unit[t] * (1.0f / kWeightScale), dacc[t]);
                f16x8 w[2];
                split_weights(phi[t][0], phi[t][1], w[0], w[1]);
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) {
                    // the third part, 2^-11 h, is formed here: reading it would be a third of the operand's bytes
                    f32x4 sum = mfma_f16(now.x[mb][0] * (_Float16)(1.0f / kWeightScale), w[1], f32x4{0.f, 0.f, 0.f, 0.f});
                    sum = mfma_f16(now.x[mb][1], w[0], sum);
                    sum = mfma_f16(now.x[mb][0], w[0], sum);
#pragma unroll
                    for (int v = 0; v < 4; ++v) tacc[t][mb][v] = fmaf(sum[v], unit[t], tacc[t][mb][v]);
                }
            }
            if (__builtin_expect(own_units, 0)) {
#pragma unroll
                for (int t = 0; t < NI; ++t)
#pragma unroll
                    for (int mb = 0; mb < KB; ++mb) tacc[t][mb] *= by[mb];
            }
        } else {
#pragma unroll
            for (int t = 0; t < NI; ++t) dacc[t] += dt[t];
        }
    };
#pragma unroll 1
    for (int at = 0; at < steps; at += DEPTH) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            if (at + k < steps) {
                chunk(chunk_at(at + k), at + k == 0, ring[k]);
                read(chunk_at(min(at + k + DEPTH, steps - 1)), ring[k]);
            }
        }
    }

    // The waves' sums.
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        float d = dacc[t];
        d += __shfl_xor(d, 16);
        d += __shfl_xor(d, 32);
        if (g == 0) sum_d[wave][t * kTile + r] = d;
    }
    if constexpr (SCORE) {
        if (HALVE) {
            if (wave >= SLOTS) {
#pragma unroll
                for (int k = 0; k < NI * KT; ++k) sum_t[wave - SLOTS][k][lane] = tacc[k / KT][k % KT];
            }
            __syncthreads();
            if (wave < SLOTS) {                     // (a lane reads and writes its own element)
#pragma unroll
                for (int k = 0; k < NI * KT; ++k) sum_t[wave][k][lane] += tacc[k / KT][k % KT];
            }
        } else {
#pragma unroll
            for (int k = 0; k < NI * KT; ++k) sum_t[wave][k][lane] = tacc[k / KT][k % KT];
        }
        __shared__ uint32_t words[FIT ? NI * kTile * (DP + 1) : 1];
        __shared__ float smean[FIT ? DP : 1];
        __shared__ uint32_t far_rows[2];
        if constexpr (FIT) {
            __shared__ int stamp_flag;
            stamp_check(out.stamp, &stamp_flag);
            if (threadIdx.x < 2) far_rows[threadIdx.x] = 0;
            if ((int)threadIdx.x < DP) smean[threadIdx.x] = (int)threadIdx.x < out.d ? out.centre[threadIdx.x] : 0.0f;
        }
        __syncthreads();
        const int item = threadIdx.x, k = item / kWave;          // this thread's output (whole waves)
        if (item < ITEMS) {
            const int of_row = k / KT * kTile + r, c0 = k % KT * 16 + g * 4;
            const int64_t i = row0 + of_row, at = i * out.d + c0;
            const bool active = i < m && c0 < out.d;
            f32x4 shifted = {0.0f, 0.0f, 0.0f, 0.0f};               // and of padding
            if (active) {
                PreparedQuad own;
                own.load(ps, i, c0, DP, kFormatHalf2, SELF ? 0 : m_pad);
                f32x4 xv = {0.0f, 0.0f, 0.0f, 0.0f};
                if (out.x_sd) xv = load_quad(out.x + at, out.quad_io, out.d - c0);
                f32x4 tsum = tree_sum<f32x4, SLOTS>([&](int q) { return sum_t[q][k][lane]; });
                const float dsum = tree_sum<float, WAVES>([&](int q) { return sum_d[q][of_row]; });
                f32x4 rest, pc = own.value(kFormatHalf2, SELF ? 0 : m_pad, &rest);
                if (__builtin_expect(other_units != 0.0f, 0)) out.units.plain(i, c0, out.d, DP, tsum, pc, rest);
                f32x4 o;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    o[v] = 0.0f;
                    if (SELF) o[v] = fmaf(-rest[v], dsum, fmaf(-pc[v], dsum, tsum[v])) / (dsum + 1.0f) * out.inv_ah2;
                    else if (dsum >= out.min_sum) o[v] = ((tsum[v] / dsum - pc[v]) - rest[v]) * out.inv_ah2;
                    shifted[v] = fmaf(out.half_h2, o[v], xv[v]);
                }
                if (out.quad_io) {
                    if (out.score) *reinterpret_cast<f32x4*>(out.score + at) = o;
                    if (out.x_sd) *reinterpret_cast<f32x4*>(out.x_sd + at) = shifted;
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (c0 + v >= out.d) break;
                        if (out.score) out.score[at + v] = o[v];
                        if (out.x_sd) out.x_sd[at + v] = shifted[v];
                    }
                }
            }
            if constexpr (FIT) {
#pragma unroll
                for (int v = 0; v < 4; ++v) words[of_row * (DP + 1) + c0 + v] = __builtin_bit_cast(uint32_t, active && c0 + v < out.d ? shifted[v] : 0.0f);
            }
        }
        if constexpr (FIT) {
            __syncthreads();
            prep_rows_half2<NI * kTile, THREADS>(out.sd_job, row0, out.d, DP, out.a, false, smean, nullptr, false, words, far_rows);
        }
    } else {
        __syncthreads();
        const int64_t i = row0 + threadIdx.x;
        if (threadIdx.x < NI * kTile && i < m) {
            const float dsum = tree_sum<float, WAVES>([&](int q) { return sum_d[q][threadIdx.x]; });
            eval_outputs(i, dsum, out.lognorm, (double)out.residual[i] * 0.69314718055994530942, LAPLACE, out.min_sum, out.density, out.log_density);
        }
    }
}

}  // namespace
