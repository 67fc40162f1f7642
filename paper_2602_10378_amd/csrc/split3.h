// Three-part bf16 operands of the fp32 mode's symmetric path: layout of the prepared arrays and the splits.
#pragma once
#include "common.h"

namespace {

// ------------------------------------------------------------------------------------------
// The symmetric path multiplies on the bf16 matrix units without giving up fp32 operands: every fp32 value v is held as
// three bf16 parts h + m + l = v (8 significant bits each; the 24 bits of v exactly, at any magnitude whose last bit
// is a normal bf16 number), and a product a b is summed over six of its nine part products,
//     ah bh + ah bm + am bh + am bm + ah bl + al bh,
// each exact in the fp32 accumulator's own format.  The three left out (am bl, al bm, al bl) are of either sign and
// together at most 2^-24 of |a b| where both operands are split to nearest (the Gram tile: |m| <= 2^-8, |l| <= 2^-17 of
// the value's power of two), the size of one fp32 rounding, and at most 1.5 2^-23 where one is truncated (the weights in
// Phi X: m < 2^-7, l < 2^-15).  Weights below about 2^-110 lose their last bits, since a bf16 part has none below 2^-133:
// less than 2^-126 of each, what the exp already flushes.  Six bf16 MFMAs per fp32 product still leave 2.6 times the
// fp32 MFMA rate.
//
// Prepared rows ("xs" / "ps"), in chunks of kChunkRows = 32 rows of KB * 3072 bytes (KB = dp / 16), two 16-row tiles of
// KB * 1536 bytes each:
//   32-column block b (columns 32b .. 32b+31): part q at b * 3072 + q * 1024; lane l = 16 g + r of the operand holds
//     columns 8g .. 8g+7 of row r at l * 16.
//   the odd 16-column block left over when KB is odd: part q at (KB / 2) * 3072 + q * 512; columns 8g .. 8g+7 (g < 2) of
//     row r at (16 g + r) * 16.  An MFMA's K = 32 then holds two parts: see read_gram in pair_split.h.
// Prepared transpose ("xt"), same chunks: 16-column block mb, part q at mb * 3072 + q * 1024; lane l = 16 g + r holds
//   column 16 mb + r of rows 4g .. 4g+3 of the first tile and 4g .. 4g+3 of the second, which is the order the Gram
//   accumulators of the two tiles leave Phi in.
// Coordinates carry the scale a sqrt 2 and norms are -|x~|^2 / 2, so that the exponent is p.x - |p|^2/2 - |x|^2/2.
// ------------------------------------------------------------------------------------------

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kChunkRows = 32;
constexpr float kBf16Max = 3.38953139e38f;       // largest finite bf16 value
constexpr int kPartBytes = 1024;                 // one part of a 16-row x 32-column operand
constexpr int chunk_bytes(int kb) { return kb * 3 * kPartBytes; }
// fp32 values needed to hold `rows` prepared rows of kb blocks (6 bytes a value)
inline int64_t split3_floats(int64_t rows, int dp) { return rows * dp * 3 / 2; }

// Byte offset of (row, column c), part 0, in the prepared rows; *part_stride: bytes from one part to the next.
__device__ __forceinline__ int64_t split3_offset(int64_t row, int c, int dp, int* part_stride)
{
    const int kb = dp / 16, r = (int)(row & 15);
    const int64_t tile = (row >> 4) * (int64_t)(kb * 1536);
    const int b = c >> 5;
    const bool odd = 2 * b + 1 >= kb;
    *part_stride = odd ? 512 : kPartBytes;
    return tile + b * 3072 + (((c >> 3) & (odd ? 1 : 3)) * 16 + r) * 16 + (c & 7) * 2;
}

__device__ __forceinline__ float bf16_value(uint16_t bits) { return __builtin_bit_cast(float, (uint32_t)bits << 16); }

// Four fp32 values from their three parts (the sums are exact).
__device__ __forceinline__ f32x4 split3_sum(const u32x2 (&part)[3])
{
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 2; q >= 0; --q)
        v += f32x4{bf16_value(part[q].x & 0xffffu), __builtin_bit_cast(float, part[q].x & 0xffff0000u),
                   bf16_value(part[q].y & 0xffffu), __builtin_bit_cast(float, part[q].y & 0xffff0000u)};
    return v;
}

// Round-to-nearest split of two values into packed bf16 parts (preparation).
__device__ __forceinline__ void split3_rne(float a, float b, uint32_t (&part)[3])
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const f32x2 v = {a, b};
        part[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
        a -= __builtin_bit_cast(float, part[q] << 16);
        b -= __builtin_bit_cast(float, part[q] & 0xffff0000u);
    }
}

// Eight weights into parts by truncation: the top 16 bits of a value are its first part, the top 16 of the remainder
// (exact) the second, of the remainder's remainder the third.  A v_perm_b32 packs two; a v_and_b32 and a v_sub_f32 per
// value form the remainder, both at the full vector rate (v_cvt_pk_bf16_f32 and shifts issue at half of it).
__device__ __forceinline__ void split3_weights(const f32x4& p, const f32x4& q, bf16x8& h, bf16x8& m, bf16x8& l)
{
    uint32_t part[3][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float a = k < 2 ? p[2 * k] : q[2 * k - 4], b = k < 2 ? p[2 * k + 1] : q[2 * k - 3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
            part[s][k] = __builtin_amdgcn_perm(ub, ua, 0x07060302);      // [high half of a | high half of b]
            if (s < 2) {
                a -= __builtin_bit_cast(float, ua & 0xffff0000u);
                b -= __builtin_bit_cast(float, ub & 0xffff0000u);
            }
        }
    }
    h = __builtin_bit_cast(bf16x8, (u32x4){part[0][0], part[0][1], part[0][2], part[0][3]});
    m = __builtin_bit_cast(bf16x8, (u32x4){part[1][0], part[1][1], part[1][2], part[1][3]});
    l = __builtin_bit_cast(bf16x8, (u32x4){part[2][0], part[2][1], part[2][2], part[2][3]});
}

// 16 bytes at a wave-uniform base plus an unsigned lane offset.  The empty asm keeps the base in scalar registers: left
// to itself the compiler adds the lane offset to a loop-invariant pointer first and carries 64-bit vector addresses.
template <typename T>
__device__ __forceinline__ T load_at(const char* base, uint32_t offset)
{
    uint64_t bits = reinterpret_cast<uint64_t>(base);
    asm("" : "+s"(bits));
    typedef const __attribute__((address_space(1))) char* global_bytes;
    return *reinterpret_cast<const __attribute__((address_space(1))) T*>(reinterpret_cast<global_bytes>(bits) + offset);
}

__device__ __forceinline__ f32x4 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x4& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace
