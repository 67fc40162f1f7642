// Prep kernels: centre + scale + pad (+ fp16 hi/lo split) into the layouts the pair kernels read.
#pragma once
#include "common.h"
#include "half2.h"
#include "split3.h"

namespace {

// ------------------------------------------------------------------------------------------
// Prep: the centre (mean of a strided subsample, formed by every workgroup for itself), then centre + scale + pad.
// ------------------------------------------------------------------------------------------

// v summed over each group of eight lanes, in all of them (lane ^ 1, lane ^ 2, then the row of eight mirrored).
__device__ __forceinline__ double sum_of_eight(double v)
{
    auto add = [](double x, auto ctrl) {
        const uint64_t bits = __builtin_bit_cast(uint64_t, x);
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)bits, decltype(ctrl)::value, 0xf, 0xf, true);
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(bits >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return x + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };
    v = add(v, std::integral_constant<int, 0xB1>());        // quad_perm [1, 0, 3, 2]
    v = add(v, std::integral_constant<int, 0x4E>());        // quad_perm [2, 3, 0, 1]
    return add(v, std::integral_constant<int, 0x141>());    // row_half_mirror
}

__device__ __forceinline__ float sum_of_eight(float v)
{
    auto add = [](float x, auto ctrl) {
        return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = add(v, std::integral_constant<int, 0xB1>());
    v = add(v, std::integral_constant<int, 0x4E>());
    return add(v, std::integral_constant<int, 0x141>());
}

// The centre all coordinates are taken relative to: the column means of an evenly strided subsample of the
// samples (about kCentreElems input values, at least 32 rows), summed in double in a fixed order, so every
// workgroup that computes it gets the same bits.  Any point near the data serves (the exponent
// -|p - x|^2 / 2h^2 does not depend on it; it only keeps the norms of the Gram expansion small), so a few hundred
// rows spread over the whole array are as good as all of them and need no pass of their own.
// Result in smean[0 .. d).
inline int64_t centre_rows(int64_t n, int d)
{
    const int64_t want = kCentreElems / d > 32 ? kCentreElems / d : 32;
    return n < want ? n : want;
}

// Where a prep launch gets the centre from.
struct PrepCommon {
    const float* centre_src;   // samples to take the centre of; null: read `centre`
    int64_t rows, stride;      // centre_rows of them, this many rows apart (>= 1)
    double weight;             // 1 / rows
    float* centre;             // in the workspace: written by workgroup 0 when computed, read otherwise
    float* units;              // the same for the units of "xt" (half2.h); null: none wanted
};
inline PrepCommon centre_of(const float* src, int64_t n, int d, float* centre, float* units)
{
    const int64_t rows = src ? centre_rows(n, d) : 1;
    return {src, rows, src ? n / rows : 1, 1.0 / (double)rows, centre, units};
}

// The unit of a column whose coordinates are about `spread` apart: 2^k that makes that 32 to 64, if it is below 1/4.
__device__ __forceinline__ float unit_of(float spread)
{
    if (!(spread > 0.0f && spread < 0.25f)) return 1.0f;   // (a constant column, or nothing known: as it is)
    const int k = 5 + 127 - (int)(__builtin_bit_cast(uint32_t, spread) >> 23);
    return __builtin_bit_cast(float, (uint32_t)(127 + (k < kMostUnit ? k : kMostUnit)) << 23);
}

// Ends with a barrier; meanwhile() is called before one, once the loads above it have been waited for.  UNITS: also the columns'
// units into sunit, from the mean difference of rows that follow each other in a thread (its first: from row 0), which needs
// no mean; *other (0, since before a barrier): whether one is not 1.
template <bool UNITS, typename F>
__device__ __forceinline__ void block_centre(const PrepCommon& pc, int d, float a, double* red, float* smean, float* sunit, uint32_t* other, F meanwhile)
{
    const int rows_per_iter = kBlock / d;                 // d <= 128 < kBlock
    const int rr = threadIdx.x / d, c = threadIdx.x % d;
    const int rows = (int)pc.rows;
    __shared__ float red_apart[UNITS ? kBlock : 1];
    double acc = 0.0;
    float apart = 0.0f;
    if (rr < rows_per_iter) {
        float before = UNITS ? pc.centre_src[c] : 0.0f;
        const float* at = pc.centre_src + rr * pc.stride * d + c;
        const int64_t step = rows_per_iter * pc.stride * d;
#pragma unroll 16
        for (int k = rr; k < rows; k += rows_per_iter) {
            const float x = *at;
            at += step;
            acc += (double)x;
            if (UNITS) apart += fabsf(x - before);
            before = x;
        }
    }
    red[threadIdx.x] = acc;
    if (UNITS) red_apart[threadIdx.x] = apart;
    meanwhile();
    __syncthreads();
    auto finish = [&](int col, double sum, float steps) {
        smean[col] = (float)(sum * pc.weight);
        if constexpr (UNITS) {
            const float unit = pc.units ? unit_of(steps * (float)pc.weight * a) : 1.0f;
            sunit[col] = unit;
            if (unit != 1.0f) *other = 1;
        }
    };
    // eight threads a column (by one the reads of its partial sums were a chain of 256 / d LDS latencies)
    if (8 * d <= kBlock) {
        const int col = threadIdx.x / 8;
        if (col < d) {
            double t = 0.0;
            float t2 = 0.0f;
#pragma unroll 4
            for (int q = threadIdx.x % 8; q < rows_per_iter; q += 8) {
                t += red[q * d + col];
                if (UNITS) t2 += red_apart[q * d + col];
            }
            t = sum_of_eight(t);
            if (UNITS) t2 = sum_of_eight(t2);
            if (threadIdx.x % 8 == 0) finish(col, t, t2);
        }
    } else if ((int)threadIdx.x < d) {
        double t = 0.0;
        float t2 = 0.0f;
#pragma unroll 4
        for (int q = 0; q < rows_per_iter; ++q) {
            t += red[q * d + threadIdx.x];
            if (UNITS) t2 += red_apart[q * d + threadIdx.x];
        }
        finish((int)threadIdx.x, t, t2);
    }
    __syncthreads();
}

// Centre into smean and (UNITS) the columns' units into sunit (computed, or the centre read back, all units 1).  Ends with a barrier.
template <bool UNITS, typename F>
__device__ __forceinline__ void prep_common(const PrepCommon& pc, int d, double a, double* red, float* smean, float* sunit, uint32_t* other, F meanwhile)
{
    if (pc.centre_src) {
        block_centre<UNITS>(pc, d, (float)a, red, smean, sunit, other, meanwhile);
        if (blockIdx.x == 0 && (int)threadIdx.x < d) pc.centre[threadIdx.x] = smean[threadIdx.x];
        if (UNITS && pc.units && blockIdx.x == 0 && threadIdx.x < SDKDE_MAX_D) {
            const int dp = (d + 15) / 16 * 16, c = threadIdx.x;
            if (c < dp) {
                pc.units[c] = c < d ? sunit[c] : 1.0f;
                pc.units[dp + 4 + c] = c < d ? smean[c] : 0.0f;
            }
            if (c == 0) {
                pc.units[dp] = *other ? 1.0f : 0.0f;
                pc.units[dp + 1] = (float)a;
                pc.units[dp + 2] = (float)(a - (double)(float)a);
            }
        }
    } else {
        if ((int)threadIdx.x < d) smean[threadIdx.x] = pc.centre[threadIdx.x];
        if (UNITS && (int)threadIdx.x < d) sunit[threadIdx.x] = 1.0f;
        meanwhile();
        __syncthreads();
    }
}

// One array to prepare: src[rows][d] -> dst (rows_pad rows), optional blocked transpose dst_t, norms dst_n.
struct PrepJob {
    const float* src;
    int64_t rows, rows_pad;
    float* dst;
    float* dst_t;
    float* dst_n;
    float pad_value;      // thin path only: coordinate value of padding rows
    bool samples;         // the rows are summed over (not only evaluated at)
    bool shifted;         // points of max-shifted sums, or samples of the scores that are such sums
    int tail;             // kFormatHalf2: half_tail of the kernel they are for
};

// Record of what a prep launch left in the workspace (sample arrays and column sums), kept in the workspace itself:
// a launch that prepares samples writes it, a launch that relies on earlier samples (SDKDE_FLAG_SAMPLES_PREPARED)
// compares it with what it expects and, on a mismatch, poisons its own outputs with NaN so that every result of the
// call is NaN instead of a plausible number from someone else's samples.
constexpr int kStampWords = 6;
struct Stamp {
    uint64_t* where;                // in the workspace; null: no record kept or checked
    int check;                      // 0: write `value` (workgroup 0), 1: compare with `value`
    uint64_t value[kStampWords];    // kind of call, samples pointer, n, d, operand format, bits of the scale a
};

// Thread 0 of every workgroup reads or (workgroup 0) writes the record; *flag, after a barrier: whether this launch is poisoned.
__device__ __forceinline__ void stamp_check(const Stamp& stamp, int* flag)
{
    if (threadIdx.x == 0) {
        int bad = 0;
        if (stamp.where && stamp.check) {
            for (int k = 0; k < kStampWords; ++k) bad |= stamp.where[k] != stamp.value[k];
        } else if (stamp.where && blockIdx.x == 0) {
            for (int k = 0; k < kStampWords; ++k) stamp.where[k] = stamp.value[k];
        }
        *flag = bad;
    }
}

constexpr int kPrepRows = 32;      // rows per workgroup of prep_mfma_kernel (two 16-sample tiles, one chunk of half2.h, split3.h)

// The input values of rows r0 .. r0 + kPrepRows of a job, on their way to words[][] (rows of dp + 1 floats): columns
// 16 k + 2 (threadIdx.x % 8) and the next of row threadIdx.x / 8 by each thread.  Loaded before the centre is known, so that the
// two latencies of a small call's first launch are one.
// COLUMNS: most there are.
template <int COLUMNS>
struct StagedRows {
    float own[2 * COLUMNS / 16];

    __device__ __forceinline__ void load(const PrepJob& job, int64_t r0, int d)
    {
        const int64_t row = r0 + (threadIdx.x >> 3);
        const float* const in = job.src + row * d;
#pragma unroll
        for (int k = 0; k < COLUMNS / 16; ++k) {
            if (16 * k >= d) break;
            const int c = 16 * k + 2 * (threadIdx.x & 7);
            own[2 * k] = row < job.rows && c < d ? in[c] : 0.0f;
            own[2 * k + 1] = row < job.rows && c + 1 < d ? in[c + 1] : 0.0f;
        }
    }
    __device__ __forceinline__ void store(float* words, int d, int dp) const
    {
        float* const at = words + (threadIdx.x >> 3) * (dp + 1) + 2 * (threadIdx.x & 7);
#pragma unroll
        for (int k = 0; k < COLUMNS / 16; ++k) {
            if (16 * k >= d) break;
            at[16 * k] = own[2 * k];
            at[16 * k + 1] = own[2 * k + 1];
        }
    }
};

// The body of prep_mfma_kernel for one workgroup and two fp16 parts a value (half2.h): rows r0 .. r0 + ROWS of `job`, by BLOCK threads.
// Their input values stand in words[][] as floats.  far_rows[2]: zeros, since before a barrier.  sunit: the columns' units, for a
// job with a dst_t, other: whether one is not 1.  Coordinates are formed as sums of two floats: what the split leaves of them is then all that is lost (one float rounded the difference and the
// product first; in double, with its conversions, a small launch took 0.8 us longer).  A launch of a few workgroups is a chain
// of latencies: kernel arguments, centre, coordinates, stores.  Rows loaded beside the centre's, eight lanes summing each
// column of the centre, one barrier less and the norms in a wave without other work: 4.9 to 4.7 us at 4096 x 1024, d = 16.
template <int ROWS, int BLOCK>
__device__ __forceinline__ void prep_rows_half2(const PrepJob& job, int64_t r0, int d, int dp, double a, bool poisoned,
                                                const float* smean, const float* sunit, bool other, uint32_t* words, uint32_t* far_rows)
{
    static_assert(ROWS == kPrepRows || ROWS == kTile, "a workgroup writes whole chunks, or tiles (of a job without a dst_t)");
    static_assert(BLOCK % kWave == 0 && BLOCK >= 8 * ROWS, "eight lanes a row");
    const int stride = dp + 1;                  // odd: columns are read without bank conflicts
    const double reach = job.samples || !job.shifted ? kReach : kFarPoint;          // largest norm held as it is
    auto coordinate = [&](int c, float in) { return a * ((double)in - (double)smean[c]); };
    const bool may_exceed = job.dst_t != nullptr && (other || job.shifted);      // the range, in a column's unit
    __shared__ double squares[ROWS];
    if (BLOCK == 8 * ROWS || threadIdx.x < 8 * ROWS) {
        const int own = threadIdx.x >> 3, lane8 = threadIdx.x & 7;
        const int64_t row = r0 + own;
        const bool live = row < job.rows;
        double square = 0.0;
        uint32_t* const at = words + own * stride;
        float most = 0.0f;                      // in the columns' units
#pragma unroll 1
        for (int c0 = 2 * lane8; c0 < dp; c0 += 16)
#pragma unroll
            for (int c = c0; c < c0 + 2; ++c) {
                Coordinate x(a, __builtin_bit_cast(float, at[c]), c < d ? smean[c] : 0.0f);
                const bool there = live && c < d, out = there && fabsf(x.v) > kHalfMax;
                if (may_exceed && there) most = fmaxf(most, fabsf(x.v) * sunit[c]);
                if (out || !there) x.v = x.low = 0.0f;
                const uint32_t word = half2_split(x.v, x.low);
                at[c] = word;
                const double held = (double)half_low(word) + (double)half_high(word);
                square = out ? (double)__builtin_inff() : fma(held, held, square);
            }
        square = sum_of_eight(square);
        const bool beyond = square > reach * reach;         // of values that are there: such rows are read again below
        if (beyond) atomicOr(far_rows, 1u << own);          // a bit each
        if (may_exceed && most > kHalfMax && (!beyond || job.shifted)) atomicOr(far_rows + 1, 1u);
        if (lane8 == 0) squares[own] = square;
    }
    __syncthreads();
    const uint32_t far = far_rows[0];
    const bool own_units = far_rows[1] != 0;
    // such rows: 2^-k times themselves (the largest coordinate then has an exponent of 10 at most, k >= 2)
    auto largest = [&](int rr) __attribute__((always_inline)) {
        double most = 0.0;
#pragma unroll 1
        for (int c = 0; c < d; ++c) {
            const double v = fabs(coordinate(c, job.src[(r0 + rr) * d + c]));
            most = v > most || v != v ? v : most;
        }
        return most;
    };
    // infinite and NaN coordinates; of a sample also what has an infinite norm
    auto finite = [&](double most) { return most <= (job.samples ? 1.0e18 : 1.7e308); };
    // 2^k and 2^-k from the exponent bits (beyond 2^1022: 2^-k is 0)
    auto far_exponent = [](double most) __attribute__((always_inline)) {
        const uint64_t e = __builtin_bit_cast(uint64_t, most) >> 52;
        return e < 1023 + 12 ? (uint64_t)(1023 + 2) : e - 10;
    };
    auto far_scale = [&](double most) __attribute__((always_inline)) { return __builtin_bit_cast(double, far_exponent(most) << 52); };
    auto far_down = [&](double most) __attribute__((always_inline)) { return __builtin_bit_cast(double, (2046 - far_exponent(most)) << 52); };
    if (__builtin_expect(far != 0, 0)) {        // the same for all threads
#pragma unroll 1
        for (int rr = 0; rr < ROWS; ++rr) {
            if (!(far >> rr & 1u)) continue;
            const double most = largest(rr);
            const double down = finite(most) ? far_down(most) : 0.0;
#pragma unroll 1
            for (int c = threadIdx.x; c < d; c += BLOCK) {
                const double v = coordinate(c, job.src[(r0 + rr) * d + c]) * down;
                words[rr * stride + c] = finite(most) ? half2_split((float)v, (float)(v - (double)(float)v)) : 0u;
            }
        }
        __syncthreads();
    }
    // What goes into the transpose of a row's column c: without the shift a far sample has no weight, an infinite value never.
    auto for_transpose = [&](int rr, int c) __attribute__((always_inline)) {
        Coordinate x(a, 0.0f, 0.0f);
        if (c < d && r0 + rr < job.rows && (!(far >> rr & 1u) || job.shifted)) x = Coordinate(a, job.src[(r0 + rr) * d + c], smean[c]);
        if (fabsf(x.v) > 1.0e18f) x.v = x.low = 0.0f;
        return x;
    };
    __shared__ float chunk_unit[SDKDE_MAX_D];
    if (__builtin_expect(own_units, 0)) {       // the same for all threads
#pragma unroll 1
        for (int c = threadIdx.x; c < dp; c += BLOCK) {
            float most = 0.0f;
#pragma unroll 1
            for (int rr = 0; rr < ROWS; ++rr) most = fmaxf(most, fabsf(for_transpose(rr, c).v));
            const double scaled = (double)most * (c < d ? sunit[c] : 1.0f);
            const uint32_t e = scaled > kHalfMax ? (uint32_t)(__builtin_bit_cast(uint64_t, scaled) >> 52) - 1023 - 14 : 0;
            chunk_unit[c] = __builtin_bit_cast(float, (127 + e) << 23);
            half2_chunk_units(job.dst, job.rows_pad, dp)[r0 / kChunkRows * dp + c] = chunk_unit[c];
        }
        __syncthreads();
    }
    const int kb = dp / 16, tail = job.tail;
    char* const rows_out = reinterpret_cast<char*>(job.dst) + r0 / kTile * half_tile_bytes(kb);
    char* const t_out = job.dst_t ? reinterpret_cast<char*>(job.dst_t) + r0 * 6 * dp : nullptr;
    if (threadIdx.x >= BLOCK - ROWS) {        // the last wave: at dp = 16 it has no other items
        const int rr = threadIdx.x - (BLOCK - ROWS);
        const int64_t row = r0 + rr;
        const uint32_t* w = words + rr * stride;
        double acc = squares[rr], scale = 1.0;
        if (__builtin_expect(far >> rr & 1u, 0)) {
            const double most = largest(rr);
            if (finite(most)) scale = far_scale(most);
            acc = 0.0;
#pragma unroll 1
            for (int c = 0; c < dp; ++c) {
                const double v = ((double)half_low(w[c]) + (double)half_high(w[c])) * scale;
                acc = fma(v, v, acc);
            }
            // not finite: a point's sums are NaN, a sample weighs nothing (with a coordinate that is NaN: NaN)
            if (!finite(most)) acc = job.samples ? most * most : (double)__builtin_nanf("");
        }
        const float norm = poisoned ? __builtin_nanf("") : row < job.rows ? -(float)(0.5 * acc) : kPadNorm;
        const double rest = -0.5 * acc - (double)norm;
        const float left = row < job.rows && fabs(rest) < 500.0 ? (float)rest : 0.0f;       // (a norm below 2^31)
        job.dst_n[row] = norm;
        half2_scale(job.dst, job.rows_pad, dp)[row] = (float)scale;
        if (job.samples) {
            const int in_wave = (BLOCK - ROWS + rr) % kWave;            // (a tile's rows are 16 lanes in a row)
            auto any = [&](bool v) { return (__builtin_amdgcn_ballot_w64(row < job.rows && v) >> (in_wave & 48) & 0xffffu) != 0; };
            const uint32_t marks = (any(norm < -0.5f * kFarPoint * kFarPoint) ? kMarkDistant : 0) |
                                   (own_units ? kMarkOwnUnits : 0);
            if (rr % kTile == 0) half2_marks(job.dst, job.rows_pad, dp)[row / kTile] = (uint8_t)marks;
        } else {
            half2_residual(job.dst, job.rows_pad, dp)[row] = left;
        }
        if (tail != kTailNone) {        // what goes into the last block's spare columns
            const int block = dp - 16, lows = tail == kTailEight ? block : block + 8;
            uint32_t e[4];
            auto half_bits = [](float v) { return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)v); };
            e[0] = half_bits(kTermFactor[0]) | half_bits(kTermFactor[1]) << 16;
            e[1] = half_bits(kTermFactor[2]) | half_bits(left * (1.0f / kResidualFactor)) << 16;
            e[2] = w[lows] >> 16 | (w[lows + 1] & 0xffff0000u);
            e[3] = w[lows + 2] >> 16 | (w[lows + 3] & 0xffff0000u);
            int stride_of;
            char* const at = tail == kTailSpare ? rows_out + half2_offset(rr, dp - 8, dp, &stride_of)
                                                : rows_out + rr / kTile * half_tile_bytes(kb) + kb / 2 * 2048 + 1024 + rr % kTile * 16;
            *reinterpret_cast<u32x4*>(at) = u32x4{e[0], e[1], tail == kTailSpare ? 0u : e[2], tail == kTailSpare ? 0u : e[3]};
        }
    }
    // eight values at a time: of one row (rows_out), then of one column (t_out).  Whole waves take one or the other (at dp = 16
    // one wave each).
    const int row_items = ROWS * dp / 8, t_items = t_out ? kb * kWave : 0;
    for (int at_item = threadIdx.x; at_item < row_items + t_items; at_item += BLOCK) {
        uint32_t word[8];
        char* at;
        int part_stride;
        const bool of_row = at_item < row_items;
        if (of_row) {
            const int rr = at_item % ROWS, c0 = at_item / ROWS * 8;
            at = rows_out + half2_offset(rr, c0, dp, &part_stride);
#pragma unroll
            for (int k = 0; k < 8; ++k) word[k] = words[rr * stride + c0 + k];
        } else {
            const int lane = at_item % kWave, mb = (at_item - row_items) / kWave;
            const int c = mb * 16 + (lane & 15), s0 = (lane >> 4) * 4;
            at = t_out + mb * 3 * kPartBytes + lane * 16;
            part_stride = kPartBytes;
#pragma unroll
            for (int k = 0; k < 8; ++k) word[k] = words[(s0 + (k & 3) + (k >> 2) * kTile) * stride + c];
            if (__builtin_expect(other || own_units || far != 0, 0)) {                 // not what the rows hold
                const float by = (c < d ? sunit[c] : 1.0f) * (own_units ? inverse_unit(chunk_unit[c]) : 1.0f);
#pragma unroll 1
                for (int k = 0; k < 8; ++k) {
                    const Coordinate x = for_transpose(s0 + (k & 3) + (k >> 2) * kTile, c);
                    const uint32_t w = half2_split(x.v * by, x.low * by);
#pragma unroll
                    for (int q = 0; q < 8; ++q) word[q] = q == k ? w : word[q];
                }
            }
        }
        u32x4 h, l, scaled;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            h[k] = (word[2 * k] & 0xffffu) | word[2 * k + 1] << 16;
            l[k] = word[2 * k] >> 16 | (word[2 * k + 1] & 0xffff0000u);
            const _Float16 s0 = (_Float16)(half_low(word[2 * k]) * (1.0f / kWeightScale)), s1 = (_Float16)(half_low(word[2 * k + 1]) * (1.0f / kWeightScale));
            scaled[k] = (uint32_t)__builtin_bit_cast(uint16_t, s0) | (uint32_t)__builtin_bit_cast(uint16_t, s1) << 16;
        }
        if (!(of_row && tail == kTailSpare && at_item / ROWS * 8 == dp - 8)) *reinterpret_cast<u32x4*>(at) = h;     // (see above)
        *reinterpret_cast<u32x4*>(at + part_stride) = l;
        if (!of_row) *reinterpret_cast<u32x4*>(at + 2 * part_stride) = scaled;
    }
}

// Centre, scale and pad for the matrix path.  A workgroup stages kPrepRows rows in LDS and writes a (x - mean), 0 in
// padding columns and rows, to dst, the same values for the second contraction to dst_t (if it is there) and
//   dst_n[row]     = -|dst[row]|^2 in double, rounded once; kPadNorm for padding rows.
// format kFormatSplit3: dst and dst_t hold three bf16 parts of each value in the layouts of split3.h (kPrepRows rows are
// one chunk of either, so a workgroup writes two contiguous blocks, 16 bytes a thread), and the norm is halved.
// fp16x2 input modes: dst[row] holds, per 16-column block, 16 fp16 "hi" values followed by 16 fp16 "lo" values with
// hi + lo = the fp32 coordinate to ~22 mantissa bits; the norm is taken of hi + lo so that it matches what the MFMA
// multiplies; dst_t[row/16][col][row%16] = the fp32 values with each 16-sample tile transposed, except
// FP16X2_ALL: dst_t holds fp16 pairs too, laid out as the A operand of the K = 32
// second contraction: for tile, column c and lane group g, eight halves [hi(4g..4g+3) | the same again]
// followed by eight halves [lo(4g..4g+3) | the same again] (twice the bytes of the fp32 layout).
// FP16X2_PHI16: dst_t holds, for tile, column c and lane group g, eight halves
// [hi(4g..4g+3) | lo(4g..4g+3)].
// The body for one workgroup and a format other than half2.h's: rows r0 .. r0 + kPrepRows of `job`, whose input values are already in
// raw[][].
__device__ __forceinline__ void prep_rows(const PrepJob& job, int64_t r0, int d, int dp, double a, int format, bool poisoned,
                                          const float* smean, float* raw_rows, float* used_rows)
{
    // kPrepRows rows of dp + 1 floats each (odd stride: columns are read without bank conflicts)
    const int stride_f = dp + 1;
    auto raw = [&](int rr) { return raw_rows + rr * stride_f; };
    auto used = [&](int rr) { return used_rows + rr * stride_f; };
    _Float16* dst_h = reinterpret_cast<_Float16*>(job.dst);
    for (int idx = threadIdx.x; idx < kPrepRows * dp; idx += kBlock) {
        const int rr = idx / dp, c = idx % dp;
        const int64_t row = r0 + rr;
        float v = 0.0f;
        if (row < job.rows && c < d) v = (float)a * (raw(rr)[c] - smean[c]);
        raw(rr)[c] = v;
        if (format == kFormatSplit3) continue;              // the parts are written below
        const _Float16 hi = (_Float16)v;
        const _Float16 lo = (_Float16)(v - (float)hi);
        _Float16* out = dst_h + row * 2 * dp + (c / 16) * 32 + (c % 16);
        out[0] = hi;
        out[16] = lo;
        used(rr)[c] = (float)hi + (float)lo;
    }
    __syncthreads();
    if (format == kFormatSplit3) {
        static_assert(kPrepRows == kChunkRows, "a workgroup writes whole chunks");
        const int kb = dp / 16;
        char* rows_out = reinterpret_cast<char*>(job.dst) + r0 * 6 * dp;
        char* t_out = job.dst_t ? reinterpret_cast<char*>(job.dst_t) + r0 * 6 * dp : nullptr;
        // eight values at a time: of one row (rows_out), then of one column (t_out).  Whole waves take one or the other
        // (at dp = 16 one wave each), the norms below are left to the last wave.
        // A coordinate too large for bf16 goes in as zero: its norm is -inf, so every weight of the sample is exactly 0 (or NaN,
        // if another coordinate is NaN).  Its parts (inf, NaN, NaN) would make the exponents NaN instead.
        auto usable = [](float v) { return fabsf(v) > kBf16Max ? 0.0f : v; };
        const int row_items = kPrepRows * dp / 8, t_items = t_out ? kb * kWave : 0;
        for (int at_item = threadIdx.x; at_item < row_items + t_items; at_item += kBlock) {
            char* at;
            int stride;
            float v[8];
            if (at_item < row_items) {
                const int rr = at_item % kPrepRows, c0 = at_item / kPrepRows * 8;
                at = rows_out + split3_offset(rr, c0, dp, &stride);
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = usable(raw(rr)[c0 + k]);
            } else {
                const int lane = at_item % kWave, mb = (at_item - row_items) / kWave;
                const int c = mb * 16 + (lane & 15), s0 = (lane >> 4) * 4;
                at = t_out + mb * 3 * kPartBytes + lane * 16;
                stride = kPartBytes;
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = usable(raw(s0 + (k & 3) + (k >> 2) * kTile)[c]);
            }
            uint32_t part[4][3];
#pragma unroll
            for (int k = 0; k < 4; ++k) split3_rne(v[2 * k], v[2 * k + 1], part[k]);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *reinterpret_cast<u32x4*>(at + q * stride) = u32x4{part[0][q], part[1][q], part[2][q], part[3][q]};
        }
    } else if (job.dst_t && format == SDKDE_PREC_FP16X2_PHI16) {
        // A operand of the K = 32 second contraction with single-fp16 weights: for tile, column c and lane group g,
        // eight halves [hi(4g..4g+3) | lo(4g..4g+3)] (the bytes of the fp32 layout)
        _Float16* base = reinterpret_cast<_Float16*>(job.dst_t) + (r0 / kTile) * (int64_t)dp * 32;
        for (int idx = threadIdx.x; idx < kPrepRows * dp * 2; idx += kBlock) {
            // idx = ((tile*dp + c)*4 + g)*8 + e
            const int e = idx % 8, g = (idx / 8) % 4, c = (idx / 32) % dp, tile = idx / (32 * dp);
            const float v = raw(tile * kTile + 4 * g + (e & 3))[c];
            const _Float16 hi = (_Float16)v;
            base[idx] = e < 4 ? hi : (_Float16)(v - (float)hi);
        }
    } else if (job.dst_t && format != SDKDE_PREC_FP16X2_ALL) {
        float* base = job.dst_t + (r0 / kTile) * (int64_t)dp * kTile;
        for (int idx = threadIdx.x; idx < kPrepRows * dp; idx += kBlock) {
            const int tile = idx / (dp * kTile), c = (idx / kTile) % dp, rr = idx % kTile;
            base[idx] = raw(tile * kTile + rr)[c];        // idx = (tile*dp + c)*16 + rr
        }
    } else if (job.dst_t) {
        _Float16* base = reinterpret_cast<_Float16*>(job.dst_t) + (r0 / kTile) * (int64_t)dp * 64;
        for (int idx = threadIdx.x; idx < kPrepRows * dp * 4; idx += kBlock) {
            // idx = ((tile*dp + c)*4 + g)*16 + e
            const int e = idx % 16, g = (idx / 16) % 4, c = (idx / 64) % dp, tile = idx / (64 * dp);
            const float v = raw(tile * kTile + 4 * g + (e & 3))[c];
            const _Float16 hi = (_Float16)v;
            base[idx] = e < 8 ? hi : (_Float16)(v - (float)hi);
        }
    }
    if (threadIdx.x >= kBlock - kPrepRows) {
        const int rr = threadIdx.x - (kBlock - kPrepRows);
        double acc = 0.0;
        const float* v = format == kFormatSplit3 ? raw(rr) : used(rr);
        // dp is a multiple of 16: sixteen reads in flight.  One at a time, the LDS latencies of dp reads are the longest
        // chain of the kernel (FP16X2 eval at 5000 x 2000, d = 128: 14.1 us, in this form 10.7).
        for (int c0 = 0; c0 < dp; c0 += 16)
#pragma unroll
            for (int c = c0; c < c0 + 16; ++c) acc += (double)v[c] * (double)v[c];
        if (format == kFormatSplit3) acc *= 0.5;
        const int64_t row = r0 + rr;
        job.dst_n[row] = poisoned ? __builtin_nanf("") : row < job.rows ? -(float)acc : kPadNorm;
    }
}

// As much LDS as the padded dimension needs: with 33 KiB for any of them four workgroups fitted a compute unit and
// a call with more than 32768 rows took a second round of them (60028 rows at d = 24: 19 us).
inline size_t prep_lds_bytes(int dp, int format)
{
    return sizeof(float) * kPrepRows * (dp + 1) * (format == kFormatSplit3 || format == kFormatHalf2 ? 1 : 2);
}

// Grid: job0's blocks first (blocks0 of them), then job1's.  HALF2: the layout is half2.h's (built apart: the formats' code together takes
// registers).
template <bool HALF2, int COLUMNS>
__global__ __launch_bounds__(kBlock) void prep_mfma_kernel(PrepJob job0, PrepJob job1, int blocks0, int d, int dp,
                                                           PrepCommon common, double a, int format, Stamp stamp)
{
    __shared__ double red[kBlock];
    __shared__ float smean[SDKDE_MAX_D], sunit[SDKDE_MAX_D];
    extern __shared__ float prep_lds[];     // prep_lds_bytes: a (x - mean), then (fp16 formats) the hi + lo multiplied instead
    __shared__ int stamp_flag;
    __shared__ uint32_t far_rows[3];        // (and whether a unit is not 1)
    const bool second = (int)blockIdx.x >= blocks0;
    const PrepJob job = second ? job1 : job0;
    const int64_t r0 = (int64_t)(blockIdx.x - (second ? blocks0 : 0)) * kPrepRows;
    StagedRows<COLUMNS> staged;
    staged.load(job, r0, d);
    if (threadIdx.x < 3) far_rows[threadIdx.x] = 0;
    stamp_check(stamp, &stamp_flag);
    prep_common<true>(common, d, a, red, smean, sunit, far_rows + 2, [&] { staged.store(prep_lds, d, dp); });
    const bool poisoned = stamp_flag != 0;
    if constexpr (HALF2) prep_rows_half2<kPrepRows, kBlock>(job, r0, d, dp, a, poisoned, smean, sunit, far_rows[2] != 0, reinterpret_cast<uint32_t*>(prep_lds), far_rows);
    else prep_rows(job, r0, d, dp, a, format, poisoned, smean, prep_lds, prep_lds + kPrepRows * (dp + 1));
}

// Thin-d variant: dst[row][d] = a (x - mean), padding rows get pad_value in every coordinate.
// One thread per padded row; same two-job grid.
__global__ __launch_bounds__(kBlock) void prep_thin_kernel(PrepJob job0, PrepJob job1, int blocks0, int d,
                                                           PrepCommon common, float a, Stamp stamp)
{
    __shared__ double red[kBlock];
    __shared__ float smean[SDKDE_MAX_D];
    __shared__ int stamp_flag;
    stamp_check(stamp, &stamp_flag);
    prep_common<false>(common, d, a, red, smean, nullptr, nullptr, [] {});
    const bool poisoned = stamp_flag != 0;
    const bool second = (int)blockIdx.x >= blocks0;
    const PrepJob& job = second ? job1 : job0;
    const int64_t row = (int64_t)(blockIdx.x - (second ? blocks0 : 0)) * kBlock + threadIdx.x;
    if (row >= job.rows_pad) return;
    for (int c = 0; c < d; ++c)
        job.dst[row * d + c] = poisoned ? __builtin_nanf("") : row < job.rows ? a * (job.src[row * d + c] - smean[c]) : job.pad_value;
}

}  // namespace
