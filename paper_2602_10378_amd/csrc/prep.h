// Prep kernels: centre + scale + pad (+ fp16 hi/lo split) into the layouts the pair kernels read.
#pragma once
#include "common.h"
#include "split3.h"

namespace {

// ------------------------------------------------------------------------------------------
// Prep: the centre (mean of a strided subsample, formed by every workgroup for itself), then centre + scale + pad.
// ------------------------------------------------------------------------------------------

// The centre all coordinates are taken relative to: the column means of an evenly strided subsample of the
// samples (about kCentreElems input values, at least 32 rows), summed in double in a fixed order, so every
// workgroup that computes it gets the same bits.  Any point near the data serves (the exponent
// -|p - x|^2 / 2h^2 does not depend on it; it only keeps the norms of the Gram expansion small), so a few hundred
// rows spread over the whole array are as good as all of them and need no pass of their own.
// Result in smean[0 .. d); ends with a barrier.
__device__ __forceinline__ int64_t centre_rows(int64_t n, int d)
{
    const int64_t want = kCentreElems / d > 32 ? kCentreElems / d : 32;
    return n < want ? n : want;
}

__device__ __forceinline__ void block_centre(const float* __restrict__ src, int64_t n, int d, double* red, float* smean)
{
    const int rows_per_iter = kBlock / d;                 // d <= 128 < kBlock
    const int rr = threadIdx.x / d, c = threadIdx.x % d;
    const int64_t rows = centre_rows(n, d);
    const int64_t stride = n / rows;                      // >= 1
    double acc = 0.0;
    if (rr < rows_per_iter) {
#pragma unroll 16
        for (int64_t k = rr; k < rows; k += rows_per_iter) acc += (double)src[k * stride * d + c];
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if ((int)threadIdx.x < d) {
        double t = 0.0;
        for (int q = 0; q < rows_per_iter; ++q) t += red[q * d + threadIdx.x];
        smean[threadIdx.x] = (float)(t / (double)rows);
    }
    __syncthreads();
}

// Where a prep launch gets the centre from.
struct PrepCommon {
    const float* centre_src;   // samples to take the centre of (centre_rows of them, strided); null: read `centre`
    int64_t centre_n;          // rows of centre_src
    float* centre;             // in the workspace: written by workgroup 0 when computed, read otherwise
};

// Centre into smean (computed or read back).  Ends with a barrier.
__device__ __forceinline__ void prep_common(const PrepCommon& pc, int d, double* red, float* smean)
{
    if (pc.centre_src) {
        block_centre(pc.centre_src, pc.centre_n, d, red, smean);
        if (blockIdx.x == 0 && (int)threadIdx.x < d) pc.centre[threadIdx.x] = smean[threadIdx.x];
    } else {
        if ((int)threadIdx.x < d) smean[threadIdx.x] = pc.centre[threadIdx.x];
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

// Thread 0 of every workgroup reads or (workgroup 0) writes the record; returns whether this launch is poisoned.
// Ends with a barrier.
__device__ __forceinline__ bool stamp_poisons(const Stamp& stamp, int* flag)
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
    __syncthreads();
    return *flag != 0;
}

constexpr int kPrepRows = 32;      // rows per workgroup of prep_mfma_kernel (two 16-sample tiles, one chunk of split3.h)

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
// The body for one workgroup: rows r0 .. r0 + kPrepRows of `job`.  STAGED: the input values of those rows are
// already in raw[][] (a caller that has just computed them); otherwise they are read from job.src.
template <bool STAGED>
__device__ __forceinline__ void prep_rows(const PrepJob& job, int64_t r0, int d, int dp, float a, int format, bool poisoned,
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
        if (row < job.rows && c < d) v = a * ((STAGED ? raw(rr)[c] : job.src[row * d + c]) - smean[c]);
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
        // A sample's coordinate too large for bf16 goes in as zero: its norm is -inf, so every weight of the sample is
        // exactly 0 (or NaN, if another coordinate is NaN).  Its parts (inf, NaN, NaN) would make the exponents NaN
        // instead.  A point keeps them: nothing can be said of its own row.
        auto usable = [&](float v) { return job.samples && fabsf(v) > kBf16Max ? 0.0f : v; };
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
    return sizeof(float) * kPrepRows * (dp + 1) * (format == kFormatSplit3 ? 1 : 2);
}

// Grid: job0's blocks first (blocks0 of them), then job1's.
__global__ __launch_bounds__(kBlock) void prep_mfma_kernel(PrepJob job0, PrepJob job1, int blocks0, int d, int dp,
                                                           PrepCommon common, float a, int format, Stamp stamp)
{
    __shared__ double red[kBlock];
    __shared__ float smean[SDKDE_MAX_D];
    extern __shared__ float prep_lds[];     // prep_lds_bytes: a (x - mean), then (fp16 formats) the hi + lo multiplied instead
    __shared__ int stamp_flag;
    const bool poisoned = stamp_poisons(stamp, &stamp_flag);
    prep_common(common, d, red, smean);

    const bool second = (int)blockIdx.x >= blocks0;
    const PrepJob& job = second ? job1 : job0;
    const int64_t r0 = (int64_t)(blockIdx.x - (second ? blocks0 : 0)) * kPrepRows;
    prep_rows<false>(job, r0, d, dp, a, format, poisoned, smean, prep_lds, prep_lds + kPrepRows * (dp + 1));
}

// Thin-d variant: dst[row][d] = a (x - mean), padding rows get pad_value in every coordinate.
// One thread per padded row; same two-job grid.
__global__ __launch_bounds__(kBlock) void prep_thin_kernel(PrepJob job0, PrepJob job1, int blocks0, int d,
                                                           PrepCommon common, float a, Stamp stamp)
{
    __shared__ double red[kBlock];
    __shared__ float smean[SDKDE_MAX_D];
    __shared__ int stamp_flag;
    const bool poisoned = stamp_poisons(stamp, &stamp_flag);
    prep_common(common, d, red, smean);
    const bool second = (int)blockIdx.x >= blocks0;
    const PrepJob& job = second ? job1 : job0;
    const int64_t row = (int64_t)(blockIdx.x - (second ? blocks0 : 0)) * kBlock + threadIdx.x;
    if (row >= job.rows_pad) return;
    for (int c = 0; c < d; ++c)
        job.dst[row * d + c] = poisoned ? __builtin_nanf("") : row < job.rows ? a * (job.src[row * d + c] - smean[c]) : job.pad_value;
}

}  // namespace
