// Symmetric score kernel: every unordered pair of samples across sample blocks once, on three-part operands.
#pragma once
#include "common.h"
#include "pair_split.h"
#include "split3.h"

namespace {

// ------------------------------------------------------------------------------------------
// Symmetric score at the samples themselves.
//
// phi_ij = phi_ji, so each unordered pair of samples needs one Gram-matrix entry, one exp and one split of the weight.
// A wave that holds row tiles I and streams sample tiles J computes the tile Phi once and uses it twice:
//   T_I^T += X_J^T (dp x 32) * Phi^T (32 x 16)     as in pair_split_kernel, Phi^T from its registers,
//   T_J^T += X_I^T (dp x 32) * Phi   (32 x 16)     with the tile's parts transposed through LDS
// (three groups of MFMAs for two ordered pairs instead of four, and half the vector work, which is more than half of
// pair_split_kernel's time at dp = 16).
//
// The samples are cut into blocks of `rb` rows; only pairs (i in an earlier block, j in a later block) are handled here,
// pairs inside one block go through pair_split_kernel restricted to that block.
// A workgroup (8 waves) takes one item = (chunk of rows c: `per_group` blocks, group gam >= c: `per_group` blocks) and,
// for every block b of the group:
//   - keeps the accumulators [T_J | D_J] of the block's rb rows in LDS ([KB][rb][16] + [rb] floats),
//   - walks over the rows of c that lie before block b, 8 * NI * 16 at a time; each wave holds NI row tiles (operands and
//     T_I, D_I in registers) and streams one eighth of the block per phase, wave w taking eighth (w + phase) mod 8, so that
//     within a phase every LDS accumulator row has one owner and the order of all additions is fixed (no atomics;
//     barriers between phases),
//   - adds the wave's T_I, D_I into partial slot gam + 1 of its rows (the same lanes add the blocks of a group one after
//     the other: first a store, then read-add-write),
//   - writes the block's LDS accumulators into partial slot c.
// A row of chunk/group rho thus receives slots 0..rho (as streamed sample, one per chunk) and rho+1..ngroups (as row, one
// per group): ngroups + 1 slots, every one written exactly once (rows that meet no later block in their own group get
// zeros).
//
// The transposed tile: every MFMA operand has its contraction index on the (lane group, register) axis and its free index
// on lane % 16.  Phi^T leaves the Gram MFMA with the sample on the former and the row on the latter, which suits T_I;
// T_J contracts over the rows.  A lane writes the four bf16 values of one part (samples 4g .. 4g+3 of row r) as 8 bytes of
// a 16 x 16 tile, ds_read_b64_tr_b16 returns rows 4g .. 4g+3 of sample r: with a second row tile's the K = 32 operand in
// the row order of the prepared transpose, which therefore serves as X_I^T as it is.
//
// Measured (clocks per 256 ordered pairs and SIMD; fp32 MFMA form before): d = 16 n = 32768 268 (317), n = 131072 221 (277),
// n = 1048576 212 (266); d = 32 n = 100000 416 (583).  Its instructions alone take about 155 at d = 16: the rest is the
// dependent chain of a pair of row tiles (Gram, weights, transposes, sums) with two waves per SIMD that meet at every phase.
// ------------------------------------------------------------------------------------------
constexpr int kSymWaves = 8;
constexpr int kSymBlock = kSymWaves * kWave;
constexpr int kSymTrBytes = 2 * 3 * 512;       // a wave's transpose buffer: two row tiles, three parts of a 16 x 16 tile

inline size_t sym_lds_bytes(int kb, int rb)
{
    return sizeof(float) * ((size_t)kb * rb * 16 + rb) + kSymWaves * kSymTrBytes;
}

// x summed over the 16 lanes that share lane / 16, in every one of them (row rotations by 8, 4, 2, 1).
__device__ __forceinline__ float sum_over_row(float x)
{
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, true));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x124, 0xf, 0xf, true));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x122, 0xf, 0xf, true));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x121, 0xf, 0xf, true));
    return x;
}

template <int KB, int NI>
__global__ __launch_bounds__(kSymBlock, 2) void pair_sym_kernel(
    const float* __restrict__ xs, const float* __restrict__ xt, const float* __restrict__ xn,
    float* __restrict__ part_t, float* __restrict__ part_d, int64_t n_pad, int rb, int nblocks, int per_group,
    int ngroups)
{
    static_assert(NI % 2 == 0, "row tiles are taken two at a time: one chunk of the prepared transpose");
    extern __shared__ __align__(16) float sym_lds[];
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    constexpr int DP = KB * 16;
    constexpr int SB = kSymWaves * NI * kTile;          // rows a workgroup holds at a time
    constexpr int PAIRS = KB / 2;
    constexpr bool ODD = KB % 2 != 0;
    constexpr int GROUPS = PAIRS + (ODD ? 1 : 0);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r = lane & 15, g = lane >> 4;
    const char* const xs_b = reinterpret_cast<const char*>(xs);
    const char* const xt_b = reinterpret_cast<const char*>(xt);
    // byte offsets of the lane, unsigned: added to a scalar base inside the load
    const uint32_t lane16 = lane * 16u, half = (16u * (g & 1) + r) * 16u, half_hl = half + (g < 2 ? 0u : 1024u), group16 = g * 16u;

    float* const lds_t = sym_lds;                            // [KB][rb][16]
    float* const lds_d = lds_t + (size_t)KB * rb * 16;       // [rb]
    char* const tr = reinterpret_cast<char*>(lds_d + rb) + wave * kSymTrBytes;      // this wave's transpose buffer
    char* const tr_wr = tr + r * 32 + g * 8;                                        // row r, samples 4g .. 4g+3
    char* const tr_rd = tr + (4 * g + (r >> 2)) * 32 + (r & 3) * 8;

    // item -> (c, gam): the ngroups (ngroups - 1) / 2 full rectangles first, the triangular items c == gam last
    const int id = blockIdx.x;
    const int noff = ngroups * (ngroups - 1) / 2;
    int c, gam;
    if (id < noff) {
        gam = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)id)) * 0.5f);
        while (gam * (gam - 1) / 2 > id) --gam;
        while ((gam + 1) * gam / 2 <= id) ++gam;
        c = id - gam * (gam - 1) / 2;
    } else {
        c = gam = id - noff;
    }
    const int b_lo = gam * per_group, b_hi = min(nblocks, b_lo + per_group);
    const int64_t a_lo = (int64_t)c * per_group * rb;
    const int64_t a_hi = min(n_pad, a_lo + (int64_t)per_group * rb);
    const int64_t slot_a = gam + 1, slot_b = c;
    const int per_phase = rb / (kSymWaves * kChunkRows);     // chunks, a power of two (host side)
    const int phase_shift = __ffs(per_phase) - 1;

    // A lane number the compiler cannot see through: address arithmetic of the code around the hot loop stays where it
    // is used instead of being hoisted into registers that the hot loop needs.
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    for (int b = b_lo; b < b_hi; ++b) {
        for (int idx = opaque(threadIdx.x); idx < KB * rb * 16 + rb; idx += kSymBlock) sym_lds[idx] = 0.0f;
        __syncthreads();
        const int bc0 = b * (rb / kChunkRows);                // first chunk of the block
        const int64_t a_end = min(a_hi, (int64_t)b * rb);     // rows strictly before the block

        for (int64_t a0 = a_lo; a0 < a_end; a0 += SB) {
            const int64_t row0 = a0 + (int64_t)wave * (NI * kTile);
            SplitRows<KB, NI> rows;
            rows.load(xs, xn, row0, opaque(r), opaque(g));
            bf16x8 xti[NI / 2][KB][3];      // T_J contraction, A: parts of column 16mb + r of the rows of two row tiles
#pragma unroll
            for (int p = 0; p < NI / 2; ++p)
#pragma unroll
                for (int mb = 0; mb < KB; ++mb)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        xti[p][mb][q] = load_at<bf16x8>(xt_b + (row0 / kChunkRows + p) * chunk_bytes(KB), (mb * 3 + q) * kPartBytes + opaque(lane) * 16u);
            f32x4 tacc[NI][KB];
            float dacc[NI];
#pragma unroll
            for (int t = 0; t < NI; ++t) {
                dacc[t] = 0.0f;
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            }

            // The wave's stream of chunks through the block: position q is chunk q % per_phase of eighth
            // (wave + q / per_phase) mod 8; at every multiple of per_phase all waves meet.
            const int q_end = kSymWaves * per_phase;
            auto chunk_of = [&](int q) {
                q = min(q, q_end - 1);                        // prefetches past the stream re-read its last chunk
                return bc0 + (((wave + (q >> phase_shift)) & (kSymWaves - 1)) << phase_shift) + (q & (per_phase - 1));
            };
            // Operands of the current chunk; each part is reloaded for the next one as soon as its last reader has issued.
            bf16x8 ga[GROUPS][2][3], ta[KB][3];
            f32x4 nj[2];
            auto load_gram = [&](int q) {
                const char* base = xs_b + (int64_t)chunk_of(q) * chunk_bytes(KB);
#pragma unroll
                for (int p = 0; p < GROUPS; ++p)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const char* at = base + u * (KB * 1536) + p * 3072;
                        if (p < PAIRS) {
#pragma unroll
                            for (int k = 0; k < 3; ++k) ga[p][u][k] = load_at<bf16x8>(at, k * kPartBytes + lane16);
                        } else {                              // [h | h], [m | m], [h | l]
                            ga[p][u][0] = load_at<bf16x8>(at, half);
                            ga[p][u][1] = load_at<bf16x8>(at, 512 + half);
                            ga[p][u][2] = load_at<bf16x8>(at, half_hl);
                        }
                    }
            };
            auto load_t = [&](int q) {
                const char* base = xt_b + (int64_t)chunk_of(q) * chunk_bytes(KB);
#pragma unroll
                for (int mb = 0; mb < KB; ++mb)
#pragma unroll
                    for (int k = 0; k < 3; ++k) ta[mb][k] = load_at<bf16x8>(base, (mb * 3 + k) * kPartBytes + lane16);
            };
            auto load_nj = [&](int q) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    nj[u] = load_at<f32x4>(reinterpret_cast<const char*>(xn + (int64_t)chunk_of(q) * kChunkRows), u * kTile * 4 + group16);
            };
            load_gram(0);
            load_nj(0);
            load_t(0);
            constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};           // Gram: largest product first
            constexpr int SA[6] = {2, 1, 0, 1, 0, 0}, SW[6] = {0, 1, 2, 0, 1, 0};           // sums: smallest first
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

#pragma unroll 1
            for (int q = 0; q < q_end; ++q) {
                f32x4 sum_j[2][KB], dj[2];          // this chunk's T_J^T (lane: columns 16mb + 4g .. +3 of sample r) and, per
                                                    // lane, the part of D_J that its row r adds to samples 4g .. 4g+3
#pragma unroll
                for (int p = 0; p < NI / 2; ++p) {
                    f32x4 cc[2][2];
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int u = 0; u < 2; ++u) cc[t][u] = nj[u] + rows.ni[2 * p + t];
#pragma unroll
                    for (int gr = 0; gr < GROUPS; ++gr)
#pragma unroll
                        for (int k = 0; k < (gr < PAIRS ? 6 : 3); ++k)
#pragma unroll
                            for (int t = 0; t < 2; ++t)
#pragma unroll
                                for (int u = 0; u < 2; ++u) {
                                    if (gr < PAIRS)
                                        cc[t][u] = mfma_bf16(ga[gr][u][PA[k]], rows.b[ODD ? 0 : 2 * p + t][PB[k]], cc[t][u]);
                                    else
                                        cc[t][u] = mfma_bf16(ga[gr][u][k < 3 ? k : 0], rows.o[ODD ? 2 * p + t : 0][k == 2 ? 1 : 0], cc[t][u]);
                                }
                    __builtin_amdgcn_sched_barrier(0);
                    if (p == NI / 2 - 1) {
                        load_gram(q + 1);
                        load_nj(q + 1);
                    }
                    bf16x8 w[2][3];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        f32x4 phi[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) phi[u][v] = __builtin_amdgcn_exp2f(cc[t][u][v]);
                            dacc[2 * p + t] += (phi[u].x + phi[u].y) + (phi[u].z + phi[u].w);
                            if (p == 0 && t == 0) dj[u] = phi[u];
                            else dj[u] += phi[u];
                        }
                        // keeps the sums here: the compiler would otherwise sink them out of the loop body's end and hold
                        // every Phi tile live
                        asm volatile("" : "+v"(dacc[2 * p + t]), "+v"(dj[0]), "+v"(dj[1]));
                        split3_weights(phi[0], phi[1], w[t][0], w[t][1], w[t][2]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    // transposed tiles of sample tile 0, then (below) of sample tile 1, through the wave's buffer
                    bf16x8 wt[2][3];
                    auto put = [&](int u) {
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                const u32x4 bits = __builtin_bit_cast(u32x4, w[t][k]);
                                *reinterpret_cast<u32x2*>(tr_wr + (t * 3 + k) * 512) = u ? u32x2{bits.z, bits.w} : u32x2{bits.x, bits.y};
                            }
                        // a wave's LDS operations execute in order: the compiler only has to keep them so
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    };
                    auto get = [&](int u) {
                        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tr_rd + k * 512)));
                            const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tr_rd + (3 + k) * 512)));
                            wt[u][k] = __builtin_bit_cast(bf16x8, (u32x4){lo.x, lo.y, hi.x, hi.y});
                        }
                    };
                    put(0);
                    get(0);
                    put(1);
                    get(1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int mb = 0; mb < KB; ++mb) {       // T_I, while the transposed tiles come back
                        f32x4 sum_i[2];
#pragma unroll
                        for (int k = 0; k < 6; ++k)
#pragma unroll
                            for (int t = 0; t < 2; ++t) sum_i[t] = mfma_bf16(ta[mb][SA[k]], w[t][SW[k]], k == 0 ? zero : sum_i[t]);
                        tacc[2 * p][mb] += sum_i[0];
                        tacc[2 * p + 1][mb] += sum_i[1];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (p == NI / 2 - 1) load_t(q + 1);
#pragma unroll
                    for (int k = 0; k < 6; ++k)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int mb = 0; mb < KB; ++mb)
                                sum_j[u][mb] = mfma_bf16(xti[p][mb][SA[k]], wt[u][SW[k]], k == 0 && p == 0 ? zero : sum_j[u][mb]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // fold the chunk's T_J and D_J into the block's accumulators
                const int row = (chunk_of(q) - bc0) * kChunkRows;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int mb = 0; mb < KB; ++mb) {
                        f32x4* at = reinterpret_cast<f32x4*>(lds_t + ((size_t)mb * rb + row + u * kTile + r) * 16 + g * 4);
                        *at += sum_j[u][mb];
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) dj[u][v] = sum_over_row(dj[u][v]);
                }
                if (r < 2) {
                    f32x4* at = reinterpret_cast<f32x4*>(lds_d + row + r * kTile + g * 4);
                    *at += r ? dj[1] : dj[0];
                }
                if (((q + 1) & (per_phase - 1)) == 0) __syncthreads();      // the same q for all waves
            }

            // this wave's rows: add into partial slot gam + 1 (the first block that meets these rows stores)
            const bool first = b == max(b_lo, (int)(a0 / rb) + 1);
            const int ro = opaque(r), go = opaque(g);
#pragma unroll
            for (int t = 0; t < NI; ++t) {
                const int64_t row = row0 + t * kTile + ro;
                float* dst = part_t + (slot_a * n_pad + row) * DP + go * 4;
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) {
                    f32x4 v = tacc[t][mb];
                    if (!first) v += *reinterpret_cast<const f32x4*>(dst + mb * 16);
                    *reinterpret_cast<f32x4*>(dst + mb * 16) = v;
                }
                float dt = dacc[t] + __shfl_xor(dacc[t], 16);
                dt += __shfl_xor(dt, 32);
                if (go == 0) {
                    float* dd = part_d + slot_a * n_pad + row;
                    *dd = first ? dt : *dd + dt;
                }
            }
        }

        // the block's accumulators -> partial slot c (every phase ended with a barrier; an empty walk leaves zeros)
        const int64_t brow = (int64_t)b * rb;
        for (int idx = opaque(threadIdx.x); idx < rb * DP; idx += kSymBlock) {
            const int j = idx / DP, col = idx % DP;
            part_t[(slot_b * n_pad + brow + j) * DP + col] = lds_t[((size_t)(col / 16) * rb + j) * 16 + (col % 16)];
        }
        for (int j = opaque(threadIdx.x); j < rb; j += kSymBlock) part_d[slot_b * n_pad + brow + j] = lds_d[j];
        __syncthreads();
    }

    // triangular item: the rows of the group's last block met no later block here; their slot gets zeros
    if (c == gam) {
        const int64_t z0 = (int64_t)(b_hi - 1) * rb;
        for (int idx = threadIdx.x; idx < rb * DP; idx += kSymBlock) part_t[(slot_a * n_pad + z0) * DP + idx] = 0.0f;
        for (int j = threadIdx.x; j < rb; j += kSymBlock) part_d[slot_a * n_pad + z0 + j] = 0.0f;
    }
}

}  // namespace
