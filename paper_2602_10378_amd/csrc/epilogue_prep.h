// One launch for two stages of the one-call pass (sdkde_fit_eval): the score epilogue at the samples themselves with
// the debiasing shift, and the preparation of the eval pass's operands (the shifted samples, which this kernel has
// just formed, and the queries).  A small problem is a chain of dependent launches and little else; this removes one.
#pragma once
#include "epilogue.h"
#include "prep.h"

namespace {

// Workgroups [0, blocks_sd): rows r0 .. r0 + kPrepRows of the samples.  The (row, four columns) items of those rows
// are reduced over the split slots exactly as score_epilogue_quad_kernel does it (64 items per pass, slots shared by
// four parts and combined in part order: the same bits), score and shifted samples are written, and the shifted
// values stay in LDS, from where prep_rows writes the eval pass's prepared copy and norms.  `ps` (the score pass's
// prepared samples, read for p~) and sd_job.dst may be the same memory: a workgroup reads its own rows before it
// overwrites them and no other workgroup touches them.
// x_sd is sd_job.src, which prep_rows reads again for samples beyond the fp16 range.
// Workgroups [blocks_sd, ...): the queries, as prep_mfma_kernel prepares them (centre read from the workspace).
template <bool HALF2>
__global__ __launch_bounds__(kBlock) void score_epilogue_prep_kernel(
    const float* __restrict__ part_t, const float* __restrict__ part_d, const float* ps, int nsplit, int64_t m,
    int64_t m_pad, int d, int dp, int any_format, float inv_ah2, float* __restrict__ score, const float* __restrict__ x,
    float half_h2, float* x_sd, int quad_io, PrepJob sd_job, PrepJob q_job, int blocks_sd,
    const float* centre, double a, Stamp stamp, ScoreUnits units)
{
    constexpr int PARTS = kEpiPartsFew, LANES = kBlock / PARTS;
    const int format = HALF2 ? kFormatHalf2 : any_format;       // (built apart, as prep_mfma_kernel)
    __shared__ float smean[SDKDE_MAX_D];
    extern __shared__ float prep_lds[];                     // prep_lds_bytes
    float* const raw = prep_lds;
    float* const used = prep_lds + kPrepRows * (dp + 1);
    __shared__ f32x4 red_t[PARTS][LANES];
    __shared__ float red_d[PARTS][LANES];
    __shared__ int stamp_flag;
    __shared__ uint32_t far_rows[2];
    if (threadIdx.x < 2) far_rows[threadIdx.x] = 0;
    const float of_centre = (int)threadIdx.x < d ? centre[threadIdx.x] : 0.0f;      // needed by prep_rows only
    const bool of_queries = (int)blockIdx.x >= blocks_sd;
    const PrepJob job = of_queries ? q_job : sd_job;
    const int64_t r0 = (int64_t)(blockIdx.x - (of_queries ? blocks_sd : 0)) * kPrepRows;
    StagedRows<32> staged;                                  // (of dp = 16)
    if (of_queries) staged.load(job, r0, d);
    stamp_check(stamp, &stamp_flag);
    if (of_queries) {
        staged.store(raw, d, dp);
    } else {
        const int lane = threadIdx.x % LANES, part = threadIdx.x / LANES;
        const int quads = dp / 4;
        for (int first = 0; first < kPrepRows * quads; first += LANES) {        // kPrepRows * quads is a multiple of 64
            const int item = first + lane;
            const int64_t i = r0 + item / quads;
            const int c0 = (item % quads) * 4;
            const bool active = i < m && c0 < d;
            f32x4 xv = {0.0f, 0.0f, 0.0f, 0.0f};
            RowSums acc = {xv, 0.0f};
            PreparedQuad prepared = {};
            const int64_t at = i * d + c0;
            if (active) {
                prepared.load(ps, i, c0, dp, format, 0);        // may run past d in the last quad: padding, not stored
                // quad_io: d is a multiple of four and the caller's arrays are 16-byte aligned
                if (part == 0) xv = load_quad(x + at, quad_io, d - c0);
                acc = sum_slots<PARTS>(part, nsplit, acc, [&](int s) {
                    return RowSums{*reinterpret_cast<const f32x4*>(part_t + ((int64_t)s * m_pad + i) * dp + c0), part_d[(int64_t)s * m_pad + i]};
                });
            }
            red_t[part][lane] = acc.t;
            red_d[part][lane] = acc.d;
            f32x4 shifted = {0.0f, 0.0f, 0.0f, 0.0f};               // and of padding
            __syncthreads();
            if (active && part == 0) {
                f32x4 tsum = tree_sum<f32x4, PARTS>([&](int k) { return red_t[k][lane]; });
                float dsum = tree_sum<float, PARTS>([&](int k) { return red_d[k][lane]; });
                f32x4 rest;
                f32x4 pc = prepared.value(format, 0, &rest);
                if (ScoreUnits::there(dsum, format)) units.plain(i, c0, d, dp, tsum, pc, rest);
                f32x4 out;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    out[v] = fmaf(-rest[v], dsum, fmaf(-pc[v], dsum, tsum[v])) / (dsum + 1.0f) * inv_ah2;   // the samples' own pair is not in the sums
#pragma unroll
                for (int v = 0; v < 4; ++v) shifted[v] = fmaf(half_h2, out[v], xv[v]);
                if (quad_io) {
                    if (score) *reinterpret_cast<f32x4*>(score + at) = out;
                    *reinterpret_cast<f32x4*>(x_sd + at) = shifted;
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (c0 + v >= d) break;
                        if (score) score[at + v] = out[v];
                        x_sd[at + v] = shifted[v];
                    }
                }
            }
            if (part == 0) {
#pragma unroll
                for (int v = 0; v < 4; ++v) raw[(item / quads) * (dp + 1) + c0 + v] = c0 + v < d ? shifted[v] : 0.0f;
            }
            __syncthreads();            // red_t / red_d are reused by the next pass; raw is read below
        }
    }
    if ((int)threadIdx.x < d) smean[threadIdx.x] = of_centre;
    __syncthreads();
    const bool poisoned = stamp_flag != 0;
    // (neither job has a dst_t)
    if constexpr (HALF2) prep_rows_half2<kPrepRows, kBlock>(job, r0, d, dp, a, poisoned, smean, nullptr, false, reinterpret_cast<uint32_t*>(raw), far_rows);
    else prep_rows(job, r0, d, dp, a, format, poisoned, smean, raw, used);
}

}  // namespace
