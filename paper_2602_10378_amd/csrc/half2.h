// Two-part fp16 operands of the fp32 path: layout of the prepared arrays and the splits.
#pragma once
#include "common.h"

namespace {

// ------------------------------------------------------------------------------------------
// The fp32 path multiplies on the fp16 matrix units.  A coordinate v = a sqrt 2 (x - mean), formed in two floats, is held as
// h + l, h = fp16(v), l = fp16(v - h), both to nearest: 11 significant bits each and a sign between them, so |v - h - l| is
// at most 2^-23 of v's power of two (0.47 of that in the root mean square; the fp32 rounding of x - mean and of its product
// with a that the second float replaces came to 0.41), or 2^-25 where |v| < 2^-2.  A product a b is summed over three of its four
// part products, ah bh + al bh + ah bl, each exact in fp32; al bl is at most 2^-22 |a b|, 2^-24.6 in the root mean square,
// of either sign.  Norms are those of h + l, so what is computed is the exact sum for samples and points moved by their
// split error, whose effect on an exponent is that error times the distance of the pair and not times the norms.
//
// Range: a sample or a point further than kReach from the centre (for the max-shifted sums a point already further than kFarPoint) is
// held as 2^-k times itself, 2^k >= 4 in the prepared `scale`, with the norm of what it stands for.  Where kernels do not ask for the
// scale it has no weight: its exponents are below -kReach^2 / 2 + kReach^2 / 4 (fp32 exponents at such distances are off by a hundred
// and more anyway).  The max-shifted sums ask for it, see pair_half.h.  Distances are norms, not single coordinates: the row's
// constant term is half a squared norm and is cut off at kLeastTerm, which has to be beyond every row that is not held so.
//
// Prepared rows ("xs" / "ps"), in chunks of kChunkRows = 32 rows, two 16-row tiles of half_tile_bytes each (KB = dp / 16):
//   32-column block b (columns 32b .. 32b+31): part q (h, l) at b * 2048 + q * 1024; lane l = 16 g + r of the operand holds
//     columns 8g .. 8g+7 of row r at l * 16.
//   the odd 16-column block left over when KB is odd, at (KB / 2) * 2048: columns 8g .. 8g+7 (g < 2) of row r, part q at
//     (32 q + 16 g + r) * 16, so that a lane's 16 bytes at (16 g + r) * 16 for g = 0 .. 3 are the K = 32 operand [h | l].
//     Behind it, at 1024 + 16 r, what fills the columns that the block's second operand (its only one, if it has at most
//     eight columns) leaves: kTermFactor, 2^7 of what rounding the norm left, and the second parts of four columns (the
//     products l l of which then are in the sum, too): columns 8 .. 11 of the block, or 0 .. 3 of eight.
//   a last 32-column block of at most 24 columns (kTailSpare): kTermFactor and the norm's residual in the first parts of columns
//     24 .. 27, zeros behind and in the second parts.
// Prepared transpose ("xt"), 2^k times the coordinates, chunks of KB * 3072 bytes: 16-column block mb, part q (h, l, 2^-11 h) at mb * 3072 + q * 1024; lane
//   16 g + r holds column 16 mb + r of rows 4g .. 4g+3 of the first tile and 4g .. 4g+3 of the second, which is the order the
//   Gram accumulators of the two tiles leave Phi in.
//   A column has a k above 0 where the coordinates are small beside 1 (less than 1/4 apart in the mean): two parts resolve 2^-25 of
//   it and no less, and a score is the small difference of sums of them.  (A column a thousand times narrower than the bandwidth:
//   its scores were good to 2 10^-5 without, 10^-7 with; one 10^6 times narrower: 2 10^-2.)  How far apart they are is seen on the
//   rows that the centre comes from, so a value can be beyond the fp16 range in such a unit: its chunk then has its own units, in
//   which its largest value has the exponent 14.
// Norms are -|h + l|^2 / 2, rounded once from double; for points `residual` holds what that rounding left.
// ------------------------------------------------------------------------------------------

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kHalfMax = 65504.0f;             // largest finite fp16 value
constexpr float kReach = 60000.0f;               // kReach^2 / 2 and the largest part of a shift beside it stay below -kLeastTerm
// From here on the shifted sums round an exponent at the size of the norms and only then shift it (its last place is 2^-3
// there): with the shift in the row's term the look for the largest exponent and the weights would miss each other, and the sums be 0
// or infinite from about 10^5 bandwidths on, with far samples from 10^4 on.
constexpr float kFarPoint = 2048.0f;
// So they do for a point that is not that far but finds nothing above this at first: its nearest sample so far is 5000 units away,
// every one more than kFarPoint from the centre.
constexpr float kFarShift = -12582912.0f;
constexpr float kWeightScale = 2048.0f;          // see pair_half.h
constexpr int half_tile_bytes(int kb) { return kb * 1024 + (kb % 2) * 256; }
// How the columns beyond whole 32-column blocks are held: none, 9 .. 16 in a 16-column block (two MFMAs), 1 .. 8 (one); 17 .. 24
// in a 32-column block whose last lane group is free for the row's term (with fewer than eight free columns the term would share
// its lane group with coordinates, whose products an MFMA then truncates at 2^-24 of the term).
enum HalfTail { kTailNone = 0, kTailSixteen = 1, kTailEight = 2, kTailSpare = 3 };
// Added in free columns instead of by four vector instructions a tile the term costs nothing but its split at the start of a row.
// Adding / in the columns of 17 to 24 of 32: eval of 10000 points against 50000 samples d = 24 110 / 100 us, d = 56 169 / 164, of
// 8000 points d = 120 258 / 250; max-shifted d = 24 178 / 154; score n = 20000 d = 56 318 / 315, n = 15000 d = 120 458 / 448.  The
// score at the samples themselves at d <= 24 adds: n = 3000 20.6 / 21.2 (the split of the term), n = 20000 within 2 %.
constexpr int half_tail(int d, bool self_score)
{
    const int last = (d - 1) % 32 + 1;
    if (self_score && d <= 24 && last > 16) return kTailNone;
    return last <= 8 ? kTailEight : last <= 16 ? kTailSixteen : last <= 24 ? kTailSpare : kTailNone;
}

// A value in two parts, the first in the low half of the word.
__device__ __forceinline__ uint32_t half2_split(float v, float low)       // v + low
{
    const _Float16 h = (_Float16)v;
    const _Float16 l = (_Float16)((v - (float)h) + low);
    return (uint32_t)__builtin_bit_cast(uint16_t, h) | (uint32_t)__builtin_bit_cast(uint16_t, l) << 16;
}
__device__ __forceinline__ float half_low(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu)); }
__device__ __forceinline__ float half_high(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16)); }

// Byte offset of (row, column c), first part, in the prepared rows; *part_stride: bytes to the second.
__device__ __forceinline__ int64_t half2_offset(int64_t row, int c, int dp, int* part_stride)
{
    const int kb = dp / 16, r = (int)(row & 15);
    const int64_t tile = (row >> 4) * (int64_t)half_tile_bytes(kb);
    const int b = c >> 5;
    const bool odd = 2 * b + 1 >= kb;
    *part_stride = odd ? 512 : 1024;
    return tile + b * 2048 + (((c >> 3) & (odd ? 1 : 3)) * 16 + r) * 16 + (c & 7) * 2;
}

// Behind the prepared points (their rows take at most 5 of the 6 bytes a value that are theirs, and dp >= 16): what rounding
// their norms left, and 2^k of points held as 2^-k times themselves.
__host__ __device__ inline float* half2_residual(float* ps, int64_t rows_pad, int dp)
{
    return ps + rows_pad / kTile * half_tile_bytes(dp / 16) / (int64_t)sizeof(float);
}
__host__ __device__ inline float* half2_scale(float* ps, int64_t rows_pad, int dp) { return half2_residual(ps, rows_pad, dp) + rows_pad; }

// Behind the prepared samples, at the same distance from them: their scales, and a byte a 16-row tile, what a kernel may have to
// know of its samples.
constexpr uint32_t kMarkDistant = 1;                // one further than kFarPoint from the centre
constexpr uint32_t kMarkOwnUnits = 2;               // its chunk's columns of "xt" are in units of their own (on both tiles of it)
constexpr uint32_t kMarks = 2;                      // how many there are
__host__ __device__ inline uint8_t* half2_marks(float* xs, int64_t rows_pad, int dp)
{
    return reinterpret_cast<uint8_t*>(half2_scale(xs, rows_pad, dp) + rows_pad);
}
// Behind the marks, for scores: the units that the columns of "xt" are in, 2^k of each of the dp columns, a float that is not 0 if any
// is not 1, the scale a in two floats, one float unused, the centre (dp floats); and for chunks with units of their own 2^e of each
// column: their values are 2^(k - e) times the coordinates.
constexpr int kMostUnit = 60;                       // k at most
__host__ __device__ inline float* half2_units(float* xs, int64_t rows_pad, int dp)
{
    return reinterpret_cast<float*>(half2_marks(xs, rows_pad, dp) + rows_pad / kTile);
}
__host__ __device__ inline float* half2_chunk_units(float* xs, int64_t rows_pad, int dp) { return half2_units(xs, rows_pad, dp) + 2 * dp + 4; }
// 2^-k of 2^k
__device__ __forceinline__ float inverse_unit(float unit) { return __builtin_bit_cast(float, 0x7f000000u - __builtin_bit_cast(uint32_t, unit)); }

// A coordinate a (x - mean) as a sum of two floats.
struct Coordinate {
    float v, low;
    __device__ __forceinline__ Coordinate(double a, float x, float mean) : Coordinate((float)a, (float)(a - (double)(float)a), x, mean) {}
    __device__ __forceinline__ Coordinate(float a_high, float a_low, float x, float mean)
    {
        const float diff = x - mean, part = diff - x, left = (x - (diff - part)) + (-mean - part);       // x - mean = diff + left
        v = a_high * diff;
        low = fmaf(a_high, diff, -v) + fmaf(a_high, left, a_low * diff);
    }
};

// The marks of chunks first .. last - 1 (and of one on either side) together, in all lanes.
__device__ __forceinline__ uint32_t marks_of(const uint8_t* marks, int first, int last, int lane)
{
    const uint32_t* const words = reinterpret_cast<const uint32_t*>(marks);     // rows are padded to 64 tiles
    uint32_t all = 0, some = 0;
    for (int w = first / 2 + lane; w * 2 < last; w += kWave) all |= words[w];
    all |= all >> 16;
    all |= all >> 8;
#pragma unroll
    for (uint32_t bit = 1; bit < 1u << kMarks; bit *= 2) some |= __builtin_amdgcn_ballot_w64((all & bit) != 0) != 0 ? bit : 0;
    return some;
}

// Four consecutive halves.
__device__ __forceinline__ f32x4 half_values(const u32x2& two)
{
    return f32x4{half_low(two.x), half_high(two.x), half_low(two.y), half_high(two.y)};
}

// The constant term of a row's exponents as three elements of a row operand: their sum with kTermFactor is the fp32 value,
// cut off where every weight is zero or no sample is within kReach (NaN stays NaN).  Each part's factor keeps it inside the fp16 range whatever v's size.
constexpr float kTermFactor[3] = {32768.0f, 16.0f, 0.0078125f};
constexpr float kLeastTerm = -kHalfMax * 32768.0f;
constexpr float kResidualFactor = 0.0078125f;       // of the samples' norms, see above
template <bool SHIFTED>
__device__ __forceinline__ void split_term(float v, float residual, _Float16 (&part)[3])
{
    v = v < kLeastTerm ? kLeastTerm : v;
    if (SHIFTED) v = v > -kLeastTerm ? -kLeastTerm : v;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (q == 2) v += residual;
        part[q] = (_Float16)(v * (1.0f / kTermFactor[q]));
        v = fmaf(-(float)part[q], kTermFactor[q], v);
    }
}

__device__ __forceinline__ f32x4 mfma_f16(const f16x8& a, const f16x8& b, const f32x4& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

}  // namespace
