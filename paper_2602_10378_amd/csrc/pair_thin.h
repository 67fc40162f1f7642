// Pair kernels of the thin path (d <= 3; the score kinds up to d = 6): direct differences on the VALU.
#pragma once
#include "common.h"
#include "prep.h"

namespace {

// ------------------------------------------------------------------------------------------
// Main pair kernel, thin-d path (Appendix A: per pair one exp and a handful of ALU ops, no
// matrix unit).  Each thread owns R evaluation rows; the streamed sample is wave-uniform, so
// its coordinates come through scalar loads.  Accumulates D_i and, for SCORE, the direct-form
// numerator N_i = sum_j phi_ij (x~_j - p~_i).  Same grid decomposition as the MFMA kernel with
// row blocks of kBlock*R rows and "tiles" of 16 samples.
// ------------------------------------------------------------------------------------------
template <int D, int R, int KIND>
__global__ __launch_bounds__(kBlock) void pair_thin_kernel(
    const float* __restrict__ ps, const float* __restrict__ xs, float* __restrict__ part_t,
    float* __restrict__ part_d, int ntiles, int tiles_per_split, int nsplit, int64_t m_pad, float laplace_c0,
    const float* __restrict__ shift)
{
    constexpr bool SCORE = KIND == kScoreSelf || KIND == kScorePoints;
    constexpr bool LAPLACE = KIND == kEvalLaplace;
    constexpr bool ROWMAX = KIND == kRowMax;
    // samples per stage: sixteen exponentials in a group for d <= 2, eight above (measured at n = 262144 with one
    // row per thread, 16 against 8: d = 1 8.5 / 9.4 ms, d = 2 12.5 / 12.6, d = 3 15.8 / 15.7, d = 6 27.3 / 26.9)
    constexpr int G = (D <= 2 ? 16 : 8) / R;
    const int split = blockIdx.x % nsplit;
    const int64_t row_block = blockIdx.x / nsplit;
    const int64_t row0 = row_block * (kBlock * R) + threadIdx.x;

    // sh[q]: the row's shift (max_j of -r^2, <= 0) in the max-shifted mode, else 0; the squared distance is
    // accumulated on top of it so that exp2(-(r^2 + sh)) = phi / 2^sh costs no extra instruction.
    // Two-level accumulation as in the matrix path: the running sums are folded into (dsum, nsum) every
    // kFlushTiles sample tiles, so that no fp32 accumulator sees a long chain of additions at its own magnitude.
    float p[R][D], dacc[R], nacc[R][SCORE ? D : 1], dsum[R], nsum[R][SCORE ? D : 1], sh[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
#pragma unroll
        for (int k = 0; k < D; ++k) p[q][k] = ps[(row0 + (int64_t)q * kBlock) * D + k];
        sh[q] = (!ROWMAX && shift) ? shift[row0 + (int64_t)q * kBlock] : 0.0f;
        dacc[q] = dsum[q] = ROWMAX ? kNegHuge : 0.0f;
#pragma unroll
        for (int k = 0; k < (SCORE ? D : 1); ++k) nacc[q][k] = nsum[q][k] = 0.0f;
    }
    auto fold = [&]() {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (ROWMAX) {
                dsum[q] = fmaxf(dsum[q], dacc[q]);
            } else {
                dsum[q] += dacc[q];
                dacc[q] = 0.0f;
            }
#pragma unroll
            for (int k = 0; k < (SCORE ? D : 1); ++k) {
                nsum[q][k] += nacc[q][k];
                nacc[q][k] = 0.0f;
            }
        }
    };

    const int t_begin = split * tiles_per_split;
    const int t_end = min(ntiles, t_begin + tiles_per_split);
    for (int jt = t_begin; jt < t_end; ++jt) {
        if (((jt - t_begin) & (kFlushTiles - 1)) == kFlushTiles - 1) fold();
        const float* xj = xs + (int64_t)jt * kTile * D;    // wave-uniform address
        // G samples at a time, in three stages pinned by scheduling barriers: squared distances, then the
        // exponentials back to back, then the sums.  v_exp_f32 issued between other VALU work slows both down
        // (measured on this chip: an exp plus four FMAs take 22.7 clocks interleaved, 20.6 in groups).
#pragma unroll
        for (int j0 = 0; j0 < kTile; j0 += G) {
            float diff[G][R][SCORE ? D : 1], r2[G][R], phi[G][R];
#pragma unroll
            for (int jj = 0; jj < G; ++jj) {
                float xv[D];
#pragma unroll
                for (int k = 0; k < D; ++k) xv[k] = xj[(j0 + jj) * D + k];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    float acc = sh[q];
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        const float df = xv[k] - p[q][k];
                        if (SCORE) diff[jj][q][k] = df;
                        acc = fmaf(df, df, acc);
                    }
                    r2[jj][q] = acc;
                }
            }
            if (ROWMAX) {
#pragma unroll
                for (int jj = 0; jj < G; ++jj)
#pragma unroll
                    for (int q = 0; q < R; ++q) dacc[q] = fmaxf(dacc[q], -r2[jj][q]);
                continue;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int jj = 0; jj < G; ++jj)
#pragma unroll
                for (int q = 0; q < R; ++q) phi[jj][q] = __builtin_amdgcn_exp2f(-r2[jj][q]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int jj = 0; jj < G; ++jj) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    // Laplace factor 1 + d/2 - r^2/2h^2, with the true r^2 = r2 - sh
                    if (LAPLACE) dacc[q] = fmaf(phi[jj][q], fmaf(sh[q] - r2[jj][q], kLn2, laplace_c0), dacc[q]);
                    else dacc[q] += phi[jj][q];
                    if (SCORE) {
#pragma unroll
                        for (int k = 0; k < D; ++k) nacc[q][k] = fmaf(phi[jj][q], diff[jj][q][k], nacc[q][k]);
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    fold();
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int64_t row = row0 + (int64_t)q * kBlock;
        part_d[(int64_t)split * m_pad + row] = dsum[q];
        if (SCORE) {
#pragma unroll
            for (int k = 0; k < D; ++k) part_t[((int64_t)split * m_pad + row) * D + k] = nsum[q][k];
        }
    }
}

// Scores on few samples: a workgroup sums 16 rows over all samples, sixteen threads a row, and writes the outputs.  A call of a few
// thousand samples is launches and little else (preparation, pairs, reduction: 13 to 45 us), and differences
// need no preparation: they are taken of the caller's values and scaled, which rounds once less than those of scaled values do.  (Not the
// eval kinds, which have to leave prepared samples behind.)  Score at the samples, three launches with split slots / this: d = 1
// n = 1000 15.4 / 9.0 us, 4000 20.4 / 9.5; d = 3 28.3 / 8.7, 30.7 / 16.2; d = 6 44.7 / 8.4, 46.3 / 21.2.  Errors against 64-bit sums
// 0.27 to 0.58 of theirs.
constexpr int kThinWholeRows = 16;
template <int D>
__global__ __launch_bounds__(kBlock) void thin_whole_kernel(
    const float* __restrict__ samples, int n, const float* __restrict__ points, int64_t m, float a, float inv_ah2, float min_sum,
    float* __restrict__ score, float half_h2, float* __restrict__ x_sd, Stamp stamp)
{
    constexpr int PARTS = kBlock / kThinWholeRows, AHEAD = 8;
    __shared__ float sums[D + 1][PARTS][kThinWholeRows + 1];
    __shared__ int stamp_flag;
    stamp_check(stamp, &stamp_flag);
    const int r = threadIdx.x % kThinWholeRows, part = threadIdx.x / kThinWholeRows;
    const int64_t row = (int64_t)blockIdx.x * kThinWholeRows + r;
    float p[D], num[D], den = 0.0f;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        p[k] = row < m ? points[row * D + k] : 0.0f;
        num[k] = 0.0f;
    }
    auto pairs = [&](int j0, auto whole) {
        float t[AHEAD][D], r2[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            const int j = j0 + q * PARTS;
            const float* const x = samples + (decltype(whole)::value || j < n ? j : 0) * (int64_t)D;
            r2[q] = 0.0f;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                t[q][k] = a * (x[k] - p[k]);
                r2[q] = fmaf(t[q][k], t[q][k], r2[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            if (!decltype(whole)::value && j0 + q * PARTS >= n) continue;
            const float phi = __builtin_amdgcn_exp2f(-r2[q]);
            den += phi;
#pragma unroll
            for (int k = 0; k < D; ++k) num[k] = fmaf(phi, t[q][k], num[k]);
        }
    };
    int j = part;
    for (; j + (AHEAD - 1) * PARTS < n; j += AHEAD * PARTS) pairs(j, std::true_type{});
    if (j < n) pairs(j, std::false_type{});
    // A sample with an infinite coordinate weighs nothing, but 0 times its difference is NaN: the numerator again without such terms
    // (in the loop above the choice is an instruction a coordinate, for samples that hardly any call has).
    bool infinite = false;
#pragma unroll
    for (int k = 0; k < D; ++k) infinite |= num[k] != num[k];
    if (__builtin_expect(infinite && den == den, 0)) {
#pragma unroll
        for (int k = 0; k < D; ++k) num[k] = 0.0f;
#pragma unroll 1
        for (j = part; j < n; j += PARTS) {
            float t[D], r2 = 0.0f;
#pragma unroll
            for (int k = 0; k < D; ++k) {
                t[k] = a * (samples[(int64_t)j * D + k] - p[k]);
                r2 = fmaf(t[k], t[k], r2);
            }
            const float phi = __builtin_amdgcn_exp2f(-r2);
#pragma unroll
            for (int k = 0; k < D; ++k) num[k] = fmaf(phi, phi == 0.0f ? 0.0f : t[k], num[k]);
        }
    }
    sums[D][part][r] = den;
#pragma unroll
    for (int k = 0; k < D; ++k) sums[k][part][r] = num[k];
    __syncthreads();
    // (D + 1) x 16 sums of sixteen parts in pairs; the first of a row's threads writes it
    for (int step = PARTS / 2; step > 0; step /= 2) {
        if (part < step) {
#pragma unroll
            for (int k = 0; k <= D; ++k) sums[k][part][r] += sums[k][part + step][r];
        }
        __syncthreads();
    }
    if (part == 0 && row < m) {
        const float dsum = sums[D][0][r];
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const float out = dsum >= min_sum ? sums[k][0][r] / dsum * inv_ah2 : 0.0f;
            if (score) score[row * D + k] = out;
            if (x_sd) x_sd[row * D + k] = fmaf(half_h2, out, p[k]);
        }
    }
}

}  // namespace
