// The symmetric score's in-block pass: both contractions on the bf16 matrix units over three-part operands.
#pragma once
#include "common.h"
#include "split3.h"

namespace {

// ------------------------------------------------------------------------------------------
// Pairs of samples inside one sample block (the pairs across blocks: pair_sym.h, whose operands these are).
// A wave owns NI tiles of 16 evaluation rows (their parts in registers, the B operand) and walks over chunks of 32
// samples (two 16-sample tiles) of its rows' block that the WAVES waves of the workgroup share through LDS.  Per (row tile, chunk):
//   C[j][i] = -|p_i|^2/2 - |x_j|^2/2 + x_j . p_i   6 KB v_mfma_f32_16x16x32_bf16 (3 KB per sample tile, fp32 accumulate)
//   Phi     = exp2(C), D_i += sum_j Phi            fp32 VALU
//   T^T    += X_J^T Phi^T                          6 KB MFMAs over the 32 samples, Phi split in registers
// The 16x16 accumulator layout (lane (r, g), register v) = (sample 4g + v, row r) is the B operand layout (k = 8g + e,
// column r) of the second contraction for the samples {4g + e of tile 0, 4g + e - 4 of tile 1}, the order in which the
// prepared transpose stores them: Phi never leaves its lane.
//
// The pair (i, i) must stay out of D and T, because T_i/D_i - x_i would otherwise cancel against the large self term whenever a
// point has few neighbours; the epilogue restores it analytically (phi_ii = 1).  In the chunks that are a wave's own rows a
// wave-uniform branch sets the diagonal's exponents to -3e38 between the Gram MFMAs and the exponentials.
//
// Grid: blockIdx.x = row block of 16 NI WAVES rows; block_tiles: sample tiles of a sample block, a multiple of the workgroup's.
// ntiles is even (host side); xs, xt, xn hold ntiles * 16 rows.
// ------------------------------------------------------------------------------------------

// Row-tile operands of one wave: -|p~|^2/2 and the parts of p~ as the lane's 16 bytes of each B operand.
template <int KB, int NI>
struct SplitRows {
    static constexpr bool ODD = KB % 2 != 0;    // one 16-column block, else one of 32 columns
    bf16x8 b[ODD ? 1 : NI][3];                  // h, m, l
    bf16x8 o[ODD ? NI : 1][2];                  // K = 32 as two parts of 16 columns: [h | m] and [l | h]
    float ni[NI];

    __device__ __forceinline__ void load(const float* __restrict__ ps, const float* __restrict__ pn, int64_t row0, int r, int g)
    {
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const char* tile = reinterpret_cast<const char*>(ps) + (row0 / kTile + t) * (int64_t)(KB * 1536);
            if (ODD) {
                const char* base = tile + (16 * (g & 1) + r) * 16;
                o[ODD ? t : 0][0] = *reinterpret_cast<const bf16x8*>(base + (g < 2 ? 0 : 512));
                o[ODD ? t : 0][1] = *reinterpret_cast<const bf16x8*>(base + (g < 2 ? 1024 : 0));
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q) b[ODD ? 0 : t][q] = *reinterpret_cast<const bf16x8*>(tile + q * kPartBytes + (16 * g + r) * 16);
            }
            ni[t] = pn[row0 + t * kTile + r];
        }
    }
};

// NB: row tiles whose Gram accumulators and split weights are live at a time.  AHEAD: operands are read from LDS a whole
// group of MFMAs before their use.
template <int KB, int NI, int WAVES, int NB, bool AHEAD, int MINW>
__global__ __launch_bounds__(WAVES * kWave, MINW) void pair_split_kernel(
    const float* __restrict__ xs, const float* __restrict__ xt, const float* __restrict__ xn, float* __restrict__ part_t,
    float* __restrict__ part_d, int ntiles, int block_tiles)
{
    static_assert(NI % 2 == 0 && NI % NB == 0, "a wave's own rows are whole chunks");
    static_assert(KB <= 2, "sums of a wave in LDS, one group of operands");
    constexpr int DP = KB * 16;
    constexpr bool ODD = KB % 2 != 0;
    constexpr int XCH = 3 * KB;                                  // 1 KiB pieces of a chunk of xs (and of xt)
    constexpr int CH = 2 * XCH;
    constexpr int STAGE = (CH + WAVES - 1) / WAVES;              // pieces a wave moves per chunk
    __shared__ __align__(16) char stage_lds[2][CH * kPartBytes];
    __shared__ f32x4 sum_lds[WAVES][NI * KB][kWave];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);    // wave-uniform by construction
    const int r = lane & 15, g = lane >> 4;
    const int64_t row_block = blockIdx.x;
    const int64_t row0 = (row_block * WAVES + wave) * (NI * kTile);

    SplitRows<KB, NI> rows;
    rows.load(xs, xn, row0, r, g);

    // Two-level accumulation: the running sums (tacc, dacc) are folded into a second level every kFlushTiles sample
    // tiles, so no fp32 accumulator sees more than a short chain of additions at its own magnitude.
    f32x4 tacc[NI][KB];
    float dacc[NI], dsum[NI];
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        dacc[t] = dsum[t] = 0.0f;
#pragma unroll
        for (int mb = 0; mb < KB; ++mb) {
            tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
            sum_lds[wave][t * KB + mb][lane] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }

    // One chunk against all NI row tiles.  own: the row tile that is the chunk's first sample tile, if it is one.
    auto chunk = [&](const char* xc, const char* tc, const f32x4& nj0, const f32x4& nj1, int own) {
        // Operands of one group of MFMAs; scheduling barriers keep an early read early.
        bf16x8 ga[2][3], ta[2][3];
        auto pin = [] { if (AHEAD) __builtin_amdgcn_sched_barrier(0); };
        auto read_gram = [&](bf16x8 (&a)[2][3]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const char* base = xc + u * (KB * 1536);
                if (!ODD) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) a[u][q] = *reinterpret_cast<const bf16x8*>(base + q * kPartBytes + lane * 16);
                } else {                            // [h | h], [m | m], [h | l]
                    const char* half = base + (16 * (g & 1) + r) * 16;
                    a[u][0] = *reinterpret_cast<const bf16x8*>(half);
                    a[u][1] = *reinterpret_cast<const bf16x8*>(half + 512);
                    a[u][2] = *reinterpret_cast<const bf16x8*>(half + (g < 2 ? 0 : 1024));
                }
            }
        };
        auto read_t = [&](int mb, bf16x8 (&a)[3]) {
#pragma unroll
            for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const bf16x8*>(tc + mb * 3072 + q * kPartBytes + lane * 16);
        };
#pragma unroll
        for (int t0 = 0; t0 < NI; t0 += NB) {
            f32x4 c[NB][2];
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                c[t][0] = nj0 + rows.ni[t0 + t];
                c[t][1] = nj1 + rows.ni[t0 + t];
            }
            read_gram(ga);
            if (AHEAD) read_t(0, ta[0]);
            pin();
            // the largest products first: they bring the accumulator from the size of the norms down to that of the distance,
            // where the small ones round finer
            if (!ODD) {
                constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int t = 0; t < NB; ++t)
#pragma unroll
                        for (int u = 0; u < 2; ++u) c[t][u] = mfma_bf16(ga[u][PA[k]], rows.b[ODD ? 0 : t0 + t][PB[k]], c[t][u]);
            } else {
                // [h | h] [h | m], [m | m] [h | m], [h | l] [l | h]
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int t = 0; t < NB; ++t)
#pragma unroll
                        for (int u = 0; u < 2; ++u) c[t][u] = mfma_bf16(ga[u][k], rows.o[ODD ? t0 + t : 0][k == 2 ? 1 : 0], c[t][u]);
            }
            pin();
            if ((unsigned)own < (unsigned)NI) {         // wave-uniform: the pairs of a point with itself
#pragma unroll
                for (int t = 0; t < NB; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (own + u == t0 + t) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) c[t][u][v] = g * 4 + v == r ? kNegHuge : c[t][u][v];
                        }
            }
            bf16x8 w[NB][3];
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                float& dt = dacc[t0 + t];
                f32x4 phi[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) phi[u][v] = __builtin_amdgcn_exp2f(c[t][u][v]);
                    dt += (phi[u].x + phi[u].y) + (phi[u].z + phi[u].w);
                }
                // keeps the sum here: the compiler would otherwise sink it behind the MFMAs and hold the Phi tiles live
                asm volatile("" : "+v"(dt));
                split3_weights(phi[0], phi[1], w[t][0], w[t][1], w[t][2]);
            }
            f32x4 sum[2][NB];
            auto add = [&](int mb) {
#pragma unroll
                for (int t = 0; t < NB; ++t) tacc[t0 + t][mb] += sum[mb & 1][t];
            };
#pragma unroll
            for (int mb = 0; mb < KB; ++mb) {
                if (!AHEAD) read_t(mb, ta[mb & 1]);
                else if (mb + 1 < KB) read_t(mb + 1, ta[(mb + 1) & 1]);
                pin();
                const bf16x8 (&a)[3] = ta[mb & 1];
                // The chunk's sum starts from zero, its smallest products first: an MFMA rounds its accumulator after
                // every lane group (four times), which this way happens at the size of 32 terms and not of the
                // running sum (summing into tacc directly: score error 1.0e-6 against 3.7e-7 at n = 32768, d = 16).
                constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int t = 0; t < NB; ++t)
                        sum[mb & 1][t] = mfma_bf16(a[PA[k]], w[t][PB[k]], k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[mb & 1][t]);
                pin();
                // added a group later, when the MFMAs have finished
                if (mb > 0) add(mb - 1);
            }
            add(KB - 1);
        }
    };

    const int own0 = (int)(row0 / kChunkRows);              // the wave's own rows are chunks own0 .. own0 + NI/2 - 1
    const int first_tile = (int)(row_block * (WAVES * NI) / block_tiles) * block_tiles;
    const int c_begin = first_tile / 2;
    const int c_end = min(ntiles, first_tile + block_tiles) / 2;
    const char* const xs_b = reinterpret_cast<const char*>(xs);
    const char* const xt_b = reinterpret_cast<const char*>(xt);
    if (c_begin < c_end) {
        const int c_last = c_end - 1;                       // the prefetch past the end re-reads the last chunk (in bounds)
        // The pieces a wave moves: both arrays advance by the same bytes per chunk, so one scalar base each (no branches
        // in the loop).  A piece past the end is the last one again, deposited twice with the same bytes.
        auto piece_of = [&](int q) { return (q + 1) * WAVES <= CH ? q * WAVES + wave : min(q * WAVES + wave, CH - 1); };
        const char* src[STAGE];
#pragma unroll
        for (int q = 0; q < STAGE; ++q) {
            const int piece = piece_of(q);                                  // wave-uniform
            src[q] = piece < XCH ? xs_b + piece * kPartBytes : xt_b + (piece - XCH) * kPartBytes;
        }
        f32x4 stage[STAGE];
        auto fetch = [&](int c) {
            const int64_t at = (int64_t)min(c, c_last) * (XCH * kPartBytes);
#pragma unroll
            for (int q = 0; q < STAGE; ++q) stage[q] = *reinterpret_cast<const f32x4*>(src[q] + at + lane * 16);
        };
        auto deposit = [&](char* buf) {
#pragma unroll
            for (int q = 0; q < STAGE; ++q) *reinterpret_cast<f32x4*>(buf + piece_of(q) * kPartBytes + lane * 16) = stage[q];
        };
        auto norms = [&](int c, int u) {
            return *reinterpret_cast<const f32x4*>(xn + (int64_t)min(c, c_last) * kChunkRows + u * kTile + g * 4);
        };
        f32x4 nj0 = norms(c_begin, 0), nj1 = norms(c_begin, 1);
        fetch(c_begin);
        deposit(stage_lds[0]);
        __syncthreads();
        for (int c = c_begin; c < c_end; ++c) {             // the same bounds for all waves of the workgroup
            const char* cur = stage_lds[(c - c_begin) & 1];
            fetch(c + 1);                                   // lands in registers while this chunk is worked on
            const f32x4 nn0 = norms(c + 1, 0), nn1 = norms(c + 1, 1);
            chunk(cur, cur + XCH * kPartBytes, nj0, nj1, 2 * (c - own0));
            if (((c + 1 - c_begin) & (kFlushTiles / 2 - 1)) == 0) {
#pragma unroll
                for (int t = 0; t < NI; ++t) {
                    dsum[t] += dacc[t];
                    dacc[t] = 0.0f;
#pragma unroll
                    for (int mb = 0; mb < KB; ++mb) {
                        sum_lds[wave][t * KB + mb][lane] += tacc[t][mb];
                        tacc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                }
            }
            nj0 = nn0;
            nj1 = nn1;
            // The other buffer was last read before the previous barrier; this barrier publishes the new chunk and
            // ends the reads of the current one.
            deposit(stage_lds[(c + 1 - c_begin) & 1]);
            __syncthreads();
        }
    }
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        const int64_t row = row0 + t * kTile + r;
#pragma unroll
        for (int mb = 0; mb < KB; ++mb)
            *reinterpret_cast<f32x4*>(part_t + row * DP + g * 4 + mb * 16) = tacc[t][mb] + sum_lds[wave][t * KB + mb][lane];
        // D needs the sum over the four lane groups g
        float dtot = dsum[t] + dacc[t];
        dtot += __shfl_xor(dtot, 16);
        dtot += __shfl_xor(dtot, 32);
        if (g == 0) part_d[row] = dtot;
    }
}

}  // namespace
