// Reductions of the partial sums and the elementwise kernels: score / eval epilogues, debias, max-shift.
#pragma once
#include "common.h"
#include "half2.h"
#include "split3.h"

namespace {

// ------------------------------------------------------------------------------------------
// Split reduction + epilogues (fixed summation order over splits: deterministic).
// ------------------------------------------------------------------------------------------

// The partial slots of one output are shared by PARTS threads (slots part, part + PARTS, ...), which keeps many
// loads in flight instead of one long dependent chain on a few compute units (a call with few points has up to
// thousands of slots and few outputs), and are combined through LDS in a fixed order (tree_sum).
// The host picks PARTS from the slot and output counts alone (epilogue_parts), so a plan always sums in the same
// order: the many-thread form only where the outputs are too few to fill the chip otherwise, since its loads are
// narrow (kBlock / PARTS consecutive floats per slot).  32 / 4 threads: 1024 outputs of 1024 slots 5.3 / 22.6 us, 4000 of
// 512 7.1 / 10.8, 8000 of 128 4.8 / 4.6, 16000 of 256 11.9 / 6.8, 18000 of 512 36.7 / 22.9, 40000 of 256 26.0 / 8.0,
// 60033 of 64 18.2 / 5.8.  (Between 8000 and the line below, the four-thread form would be 0.2 to 5 us ahead.)
constexpr int kEpiPartsFew = 4, kEpiPartsMany = 32;
constexpr int kEpiManySlots = 64;                   // least slot count and
constexpr int64_t kEpiFewOutputs = 16384;           // most outputs for kEpiPartsMany
inline int epilogue_parts(int nslots, int64_t outputs)
{
    return nslots >= kEpiManySlots && outputs <= kEpiFewOutputs ? kEpiPartsMany : kEpiPartsFew;
}

// Sum of N (a power of two) elements in pairs.  T is a sum most of which cancels against p~ D, and what adding its parts one
// after the other rounds is most of a score's error: 32 parts of 72 slots 1.7 times the error that they give in pairs (9000 samples x 300
// points, d = 9 .. 33; the same time), sixteen waves' sums in pair_whole.h 1.3 times (n = 600 .. 2000, d = 8 .. 24).
template <typename T, int N, typename F>
__device__ __forceinline__ T tree_sum(F element)
{
    T v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = element(q);
#pragma unroll
    for (int step = N / 2; step > 0; step /= 2)
#pragma unroll
        for (int q = 0; q < step; ++q) v[q] += v[q + step];
    return v[0];
}

// Slots part, part + PARTS, ... of an output: four at a time in pairs, their loads in flight together (512 slots of 1024 queries 4.8 us,
// one at a time 11.6).  One after the other, and the parts likewise, a score's error is 1.04 to 1.08 times as large (4096 .. 32768 samples,
// d = 8 .. 64).  slot(s): a sum of any kind.
template <int PARTS, typename T, typename F>
__device__ __forceinline__ T sum_slots(int part, int nslots, T acc, F slot)
{
    int s = part;
    for (; s + 3 * PARTS < nslots; s += 4 * PARTS) {
        const T v0 = slot(s), v1 = slot(s + PARTS), v2 = slot(s + 2 * PARTS), v3 = slot(s + 3 * PARTS);
        acc += (v0 + v1) + (v2 + v3);
    }
    if (s + PARTS < nslots) {
        const T v0 = slot(s), v1 = slot(s + PARTS);
        acc += v0 + v1;
        s += 2 * PARTS;
    }
    if (s < nslots) acc += slot(s);
    return acc;
}

// T (four columns) and D of a row.
struct RowSums {
    f32x4 t;
    float d;
    __device__ __forceinline__ RowSums operator+(const RowSums& o) const { return {t + o.t, d + o.d}; }
    __device__ __forceinline__ RowSums& operator+=(const RowSums& o) { return *this = *this + o; }
};

template <int PARTS, bool MAX>
__device__ __forceinline__ float reduce_slots(const float* __restrict__ first, int64_t stride, int nslots, bool active,
                                              float (*red)[kBlock / PARTS])
{
    constexpr int OUTPUTS = kBlock / PARTS;
    const int lane = threadIdx.x % OUTPUTS, part = threadIdx.x / OUTPUTS;
    float acc = MAX ? kNegHuge : 0.0f;
    if (active) {
        if constexpr (MAX) {
#pragma unroll 4
            for (int s = part; s < nslots; s += PARTS) acc = fmaxf(acc, first[(int64_t)s * stride]);
        } else {
            acc = sum_slots<PARTS>(part, nslots, 0.0f, [&](int s) { return first[(int64_t)s * stride]; });
        }
    }
    red[part][lane] = acc;
    __syncthreads();
    float r;
    if constexpr (MAX) {
        r = red[0][lane];
#pragma unroll
        for (int q = 1; q < PARTS; ++q) r = fmaxf(r, red[q][lane]);
    } else {
        r = tree_sum<float, PARTS>([&](int q) { return red[q][lane]; });
    }
    __syncthreads();            // red is reused by the next reduction
    return r;
}

// The max-shifted sums of the two-part format come with a shift of their own in every slot (pair_half.h): they are added as what they
// are of the largest one.  2^(shift - most) of a slot, both integers, 0 for a slot without samples.
__device__ __forceinline__ float slot_weight(float shift, float most) { return ldexpf(1.0f, (int)fmaxf(shift - most, -1000.0f)); }

template <int PARTS>
__device__ __forceinline__ float reduce_shifted_slots(const float* __restrict__ first, int64_t stride, const float* __restrict__ shifts, int64_t shift_stride,
                                                      float most, int nslots, bool active, float (*red)[kBlock / PARTS])
{
    constexpr int OUTPUTS = kBlock / PARTS;
    const int lane = threadIdx.x % OUTPUTS, part = threadIdx.x / OUTPUTS;
    float acc = 0.0f;
    if (active)
        acc = sum_slots<PARTS>(part, nslots, 0.0f, [&](int s) { return first[(int64_t)s * stride] * slot_weight(shifts[(int64_t)s * shift_stride], most); });
    red[part][lane] = acc;
    __syncthreads();
    const float r = tree_sum<float, PARTS>([&](int q) { return red[q][lane]; });
    __syncthreads();            // red is reused by the next reduction
    return r;
}

// Columns c0 .. c0+3 of prepared row i, in any of the formats.  The loads are asked for apart from their use, without a
// branch, so that a kernel can have them in flight beside the split slots it sums (read after the sums they are one more
// memory latency of a kernel that is little else).  scaled_rows (not 0: their padded count): points, whose rows may be held
// scaled down (half2.h).
struct PreparedQuad {
    u32x2 part[3];
    float scale;

    __device__ __forceinline__ void load(const float* ps, int64_t i, int c0, int dp, int format, int64_t scaled_rows)
    {
        int stride = 32;
        const int64_t offset = format == kFormatSplit3  ? split3_offset(i, c0, dp, &stride)
                               : format == kFormatHalf2 ? half2_offset(i, c0, dp, &stride)
                                                        : (i * 2 * dp + (c0 / 16) * 32 + c0 % 16) * 2;      // fp16 hi, lo
        const char* const at = reinterpret_cast<const char*>(ps) + offset;
        part[0] = *reinterpret_cast<const u32x2*>(at);
        part[1] = *reinterpret_cast<const u32x2*>(at + stride);
        part[2] = *reinterpret_cast<const u32x2*>(at + (format == kFormatSplit3 ? 2 * stride : 0));
        scale = *(format == kFormatHalf2 && scaled_rows ? half2_scale(const_cast<float*>(ps), scaled_rows, dp) + i
                                                        : reinterpret_cast<const float*>(at));
    }
    // The values, as a sum of two where that is more than a float holds.
    __device__ __forceinline__ f32x4 value(int format, int64_t scaled_rows, f32x4* rest) const
    {
        *rest = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (format == kFormatSplit3) return split3_sum(part);
        f32x4 v = half_values(part[0]), low = half_values(part[1]);
        if (format != kFormatHalf2) return v + low;
        if (scaled_rows) {
            v *= scale;
            low *= scale;
        }
        *rest = low;
        return v;
    }
};

// Up to four values of a row, `left` of them there; as_quad: a multiple of four are, at a multiple of 16 bytes.
__device__ __forceinline__ f32x4 load_quad(const float* at, int as_quad, int left)
{
    if (as_quad) return *reinterpret_cast<const f32x4*>(at);
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (k < left) v[k] = at[k];
    return v;
}

// What the sums T of the two-part format are in where a column has a unit of its own (half2.h); the sums D are then below zero, which
// tells the epilogues without another read.  Of such a column p~ is formed anew from the caller's array, since the prepared one
// resolves no more than 2^-25; of others the prepared one is better (what its split leaves moved the weights, too, and cancels).
// (The code for this costs score_epilogue_quad_kernel 1.1 us on small calls, 3.7 / 4.8 us at 2048 x 64, whether as a branch or
// without one, the units read early, late or not at all.)
struct ScoreUnits {
    const float* units;        // behind the prepared samples
    const float* rows;         // the points, or the samples

    __device__ __forceinline__ static bool there(float& dsum, int format)
    {
        const bool below = format == kFormatHalf2 && dsum < 0.0f;
        dsum = below ? -dsum : dsum;
        return __builtin_expect(below, 0);
    }
    __device__ __forceinline__ void plain(int64_t i, int c, int d, int dp, float& t, float& p, float& rest) const
    {
        const float unit = units[c];
        if (unit == 1.0f) return;
        const Coordinate own(units[dp + 1], units[dp + 2], rows[i * d + c], units[dp + 4 + c]);
        t *= inverse_unit(unit);
        p = own.v;
        rest = own.low;
    }
    // (a loop, so that this rare code is short)
    __device__ __forceinline__ void plain(int64_t i, int c0, int d, int dp, f32x4& t, f32x4& p, f32x4& rest) const
    {
#pragma unroll 1
        for (int v = 0; v < 4; ++v) {
            float tv = t.x, pv = p.x, rv = rest.x;
            if (c0 + v < d) plain(i, c0 + v, d, dp, tv, pv, rv);
            t = f32x4{t.y, t.z, t.w, tv};
            p = f32x4{p.y, p.z, p.w, pv};
            rest = f32x4{rest.y, rest.z, rest.w, rv};
        }
    }
};

// mode 0 (MFMA path, separate points): score = (T/D - p~) * inv_ah2            (T = Phi X regrouping)
// mode 1 (thin path):                   score = (N/D) * inv_ah2                (direct-form numerator)
// mode 2 (MFMA path, at the samples):   score = (T' - p~ D') / (D' + 1) * inv_ah2
//        where T', D' exclude the pair (i, i), whose weight is exactly 1.
// inv_ah2 = 1 / (a h^2) undoes the coordinate scaling.  D < min_sum (least_trusted_sum of the sample count) gives 0.
// score and x_sd are both optional outputs; x_sd = x + half_h2 * score (x: the original points, same indexing).
// SHIFTED: part_shift holds a shift a slot and row, [nsplit][m_pad].
// Grid: one workgroup per kBlock / PARTS elements of the [m, d] output.
template <int PARTS, bool SHIFTED>
__global__ __launch_bounds__(kBlock) void score_epilogue_kernel(
    const float* __restrict__ part_t, const float* __restrict__ part_d, const float* __restrict__ ps,
    int nsplit, int64_t m, int64_t m_pad, int d, int dp, int mode, int format, float inv_ah2,
    float* __restrict__ score, const float* __restrict__ x, float half_h2, float* __restrict__ x_sd, float min_sum, ScoreUnits units,
    const float* __restrict__ part_shift)
{
    constexpr int kEpiOutputs = kBlock / PARTS;
    __shared__ float red[PARTS][kEpiOutputs];
    const int64_t idx = (int64_t)blockIdx.x * kEpiOutputs + threadIdx.x % kEpiOutputs;
    const bool active = idx < m * d;
    const int64_t i = active ? idx / d : 0;
    const int c = active ? (int)(idx % d) : 0;
    PreparedQuad own = {};
    if (mode != 1) own.load(ps, i, c & ~3, dp, format, mode == 0 ? m_pad : 0);
    float tsum, dsum;
    if constexpr (SHIFTED) {
        const float most = reduce_slots<PARTS, true>(part_shift + i, m_pad, nsplit, active, red);
        tsum = reduce_shifted_slots<PARTS>(part_t + i * dp + c, m_pad * dp, part_shift + i, m_pad, most, nsplit, active, red);
        dsum = reduce_shifted_slots<PARTS>(part_d + i, m_pad, part_shift + i, m_pad, most, nsplit, active, red);
    } else {
        tsum = reduce_slots<PARTS, false>(part_t + i * dp + c, m_pad * dp, nsplit, active, red);
        dsum = reduce_slots<PARTS, false>(part_d + i, m_pad, nsplit, active, red);
    }
    if (!active || threadIdx.x >= kEpiOutputs) return;
    const bool in_units = ScoreUnits::there(dsum, format);
    float pc = 0.0f, rest = 0.0f;
    if (mode != 1) {
        f32x4 low;
        pc = own.value(format, mode == 0 ? m_pad : 0, &low)[c & 3];
        rest = low[c & 3];
        if (in_units) units.plain(i, c, d, dp, tsum, pc, rest);
    }
    float out = 0.0f;
    if (mode == 2) {
        out = fmaf(-rest, dsum, fmaf(-pc, dsum, tsum)) / (dsum + 1.0f) * inv_ah2;
    } else if (dsum >= min_sum) {
        float ratio = tsum / dsum;
        out = (mode == 1 ? ratio : (ratio - pc) - rest) * inv_ah2;
    }
    if (score) score[idx] = out;
    if (x_sd) x_sd[idx] = fmaf(half_h2, out, x[idx]);      // fused debiasing shift (sdkde_fit_eval)
}

// Matrix-path form of score_epilogue_kernel<kEpiPartsFew> (modes 0 and 2): a thread takes four consecutive
// coordinates of one row, so the partial T is read with 16-byte loads (1 KiB per wave and slot instead of 256
// bytes) by a quarter of the workgroups.  Same summation order, hence the same bits.  quad_io: the outputs (and x)
// may be accessed 16 bytes at a time.
// Grid: one workgroup per kBlock / kEpiPartsFew (row, four columns) pairs of the [m, d] outputs.
template <bool SHIFTED, bool HALF2>
__global__ __launch_bounds__(kBlock) void score_epilogue_quad_kernel(
    const float* __restrict__ part_t, const float* __restrict__ part_d, const float* __restrict__ ps,
    int nsplit, int64_t m, int64_t m_pad, int d, int dp, int mode, int any_format, float inv_ah2,
    float* __restrict__ score, const float* __restrict__ x, float half_h2, float* __restrict__ x_sd, int quad_io,
    float min_sum, ScoreUnits units, const float* __restrict__ part_shift)
{
    constexpr int PARTS = kEpiPartsFew, LANES = kBlock / PARTS;
    const int format = HALF2 ? kFormatHalf2 : any_format;       // (built apart: the formats' code together takes registers and time)
    __shared__ f32x4 red_t[PARTS][LANES];
    __shared__ float red_d[PARTS][LANES];
    const int lane = threadIdx.x % LANES, part = threadIdx.x / LANES;
    const int quads = (d + 3) / 4;
    const int64_t q = (int64_t)blockIdx.x * LANES + lane;
    const bool active = q < m * quads;
    const int64_t i = active ? q / quads : 0;
    const int c0 = active ? (int)(q % quads) * 4 : 0;
    const int64_t at = i * d + c0;
    PreparedQuad own;
    own.load(ps, i, c0, dp, format, mode == 0 ? m_pad : 0);       // may run past d in the last quad: padding, not stored
    f32x4 xv = {0.0f, 0.0f, 0.0f, 0.0f};
    if (x_sd && part == 0) xv = load_quad(x + at, quad_io, d - c0);
    [[maybe_unused]] float most = kNegHuge;
    if constexpr (SHIFTED) {
        if (active) {
#pragma unroll 4
            for (int s = part; s < nsplit; s += PARTS) most = fmaxf(most, part_shift[(int64_t)s * m_pad + i]);
        }
        red_d[part][lane] = most;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PARTS; ++k) most = fmaxf(most, red_d[k][lane]);
        __syncthreads();
    }
    RowSums acc = {{0.0f, 0.0f, 0.0f, 0.0f}, 0.0f};
    if (active) {
        acc = sum_slots<PARTS>(part, nsplit, acc, [&](int s) {
            const f32x4 t = *reinterpret_cast<const f32x4*>(part_t + ((int64_t)s * m_pad + i) * dp + c0);
            const float dd = part_d[(int64_t)s * m_pad + i];
            if constexpr (!SHIFTED) return RowSums{t, dd};
            const float by = slot_weight(part_shift[(int64_t)s * m_pad + i], most);
            return RowSums{t * by, dd * by};
        });
    }
    red_t[part][lane] = acc.t;
    red_d[part][lane] = acc.d;
    __syncthreads();
    if (!active || part != 0) return;
    f32x4 tsum = tree_sum<f32x4, PARTS>([&](int k) { return red_t[k][lane]; });
    float dsum = tree_sum<float, PARTS>([&](int k) { return red_d[k][lane]; });
    f32x4 rest;
    f32x4 pc = own.value(format, mode == 0 ? m_pad : 0, &rest);
    if (ScoreUnits::there(dsum, format)) units.plain(i, c0, d, dp, tsum, pc, rest);
    f32x4 out;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float o = 0.0f;
        if (mode == 2) o = fmaf(-rest[v], dsum, fmaf(-pc[v], dsum, tsum[v])) / (dsum + 1.0f) * inv_ah2;
        else if (dsum >= min_sum) o = ((tsum[v] / dsum - pc[v]) - rest[v]) * inv_ah2;
        out[v] = o;
    }
    if (quad_io) {                  // d is a multiple of four and the caller's arrays are 16-byte aligned
        if (score) *reinterpret_cast<f32x4*>(score + at) = out;
        if (x_sd) {
            f32x4 r;
#pragma unroll
            for (int v = 0; v < 4; ++v) r[v] = fmaf(half_h2, out[v], xv[v]);
            *reinterpret_cast<f32x4*>(x_sd + at) = r;
        }
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (c0 + v >= d) break;
            if (score) score[at + v] = out[v];
            if (x_sd) x_sd[at + v] = fmaf(half_h2, out[v], xv[v]);
        }
    }
}

// log p = log D + lognorm, lognorm = -log n - d log h - (d/2) log 2 pi (formed on the host in double); shift_ln: what the weights
// were divided by, as a logarithm.  is_signed (Laplace-corrected sum, which may be negative): density = sum * exp(lognorm) only.
__device__ __forceinline__ void eval_outputs(int64_t i, float dsum, double lognorm, double shift_ln, bool is_signed, float min_sum,
                                             float* __restrict__ density, float* __restrict__ log_density)
{
    // too close to the flush threshold of the weights: the all-underflow case (the signed sum of the Laplace-corrected
    // estimate may be small because its terms cancel, and is left as it is)
    if (!is_signed && dsum < min_sum) dsum = 0.0f;
    if (is_signed) {
        if (density) density[i] = (float)((double)dsum * exp(lognorm + shift_ln));
        return;
    }
    const double lp = log((double)dsum) + lognorm + shift_ln;      // -inf when dsum == 0
    if (log_density) log_density[i] = (float)lp;
    // beside the logarithm instead of after it where neither end of the double range is near (the float is 0 or inf there)
    if (density) density[i] = (float)(fabs(lognorm + shift_ln) < 600.0 ? (double)dsum * exp(lognorm + shift_ln) : exp(lp));
}

// shift (may be null): per-query base-2 exponent shift of the max-shifted mode; SHIFTED: one a slot and query, [nsplit][m_pad].
// residual (may be null): half2.h.  min_sum: least_trusted_sum(n).
// Grid: one workgroup per kBlock / PARTS queries.
template <int PARTS, bool SHIFTED>
__global__ __launch_bounds__(kBlock) void eval_epilogue_kernel(const float* __restrict__ part_d, int nsplit,
                                                               int64_t m, int64_t m_pad, double lognorm, int is_signed,
                                                               const float* __restrict__ shift,
                                                               const float* __restrict__ residual, float min_sum,
                                                               float* __restrict__ density,
                                                               float* __restrict__ log_density)
{
    constexpr int kEpiOutputs = kBlock / PARTS;
    __shared__ float red[PARTS][kEpiOutputs];
    const int64_t i = (int64_t)blockIdx.x * kEpiOutputs + threadIdx.x % kEpiOutputs;
    const bool active = i < m;
    // max-shifted mode: the sums were taken of phi / 2^shift; residual: what rounding -|p~|^2 / 2 left
    // (read from somewhere in any case: behind a branch their latency would come on top of that of the sums)
    const float* const sums = part_d + (active ? i : 0);
    float of_shift = *(shift && active ? shift + i : sums), of_residual = *(residual && active ? residual + i : sums);
    float dsum;
    if constexpr (SHIFTED) {
        const float* const shifts = shift + (active ? i : 0);
        of_shift = reduce_slots<PARTS, true>(shifts, m_pad, nsplit, active, red);
        dsum = reduce_shifted_slots<PARTS>(sums, m_pad, shifts, m_pad, of_shift, nsplit, active, red);
    } else {
        dsum = reduce_slots<PARTS, false>(sums, m_pad, nsplit, active, red);
    }
    if (!active || threadIdx.x >= kEpiOutputs) return;
    const double shift_ln = ((shift ? (double)of_shift : 0.0) + (residual ? (double)of_residual : 0.0)) * 0.69314718055994530942;
    eval_outputs(i, dsum, lognorm, shift_ln, is_signed != 0, min_sum, density, log_density);
}

// out may alias x or s (each thread reads its one element before it writes it): no __restrict__ here.
__global__ __launch_bounds__(kBlock) void debias_kernel(const float* x, const float* s, int64_t total, float half_h2,
                                                        float* out)
{
    int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (idx < total) out[idx] = fmaf(half_h2, s[idx], x[idx]);
}


// shift[i] = max over splits of the row maxima left in part_d by a kRowMax pass (thin path, fp16 input modes); on the MFMA path the
// shift is also folded into the row constant pn (-|p~|^2 - shift), so the main pass needs no extra work.
// Grid: one workgroup per kBlock / PARTS rows.
template <int PARTS>
__global__ __launch_bounds__(kBlock) void shift_kernel(const float* __restrict__ part_d, int nsplit, int64_t m_pad,
                                                       float* __restrict__ shift, float* __restrict__ pn)
{
    constexpr int kEpiOutputs = kBlock / PARTS;
    __shared__ float red[PARTS][kEpiOutputs];
    const int64_t i = (int64_t)blockIdx.x * kEpiOutputs + threadIdx.x % kEpiOutputs;
    const bool active = i < m_pad;
    // read from somewhere in any case, see eval_epilogue_kernel
    const float* const maxima = part_d + (active ? i : 0);
    const float before = *(pn && active ? pn + i : maxima);
    const float mx = reduce_slots<PARTS, true>(maxima, m_pad, nsplit, active, red);
    if (!active || threadIdx.x >= kEpiOutputs) return;
    shift[i] = pn && before == kPadNorm ? 0.0f : mx;        // a padding row's is of no interest
    if (pn) pn[i] = before - mx;
}

}  // namespace
