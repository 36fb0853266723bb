// Centroid lookup for prefill (Section 4.1) in one launch and one product per (token, cluster): a workgroup takes 32 tokens of a
// (sequence, head) and ALL of its clusters, whose scores stay in registers from the products to the decision, so neither a second
// pass over the centroids nor anything in memory between the two is needed.
//
//   per-query selection   keep cluster i for token t iff N_i > 0 and exp(x_i - m) > T * D, compared as x_i >= the least score that
//                         passes (lk_least_kept); mask words and, if asked for, the tokens' key counts.
//   MEAN                  selection on averaged scores (Appendix D, "Prefill Stage"), first half: sum over the workgroup's tokens
//                         of S_i(t) = exp(x_i - m) / D, one partial sum per cluster and part of the tokens (part_sum [B*H,
//                         n_part, C]); the selection adds the parts.  A workgroup takes token blocks part, part + n_part, ...
//
// Scores come from 32x32x16 fp16 products.  A wave owns tiles of 32 clusters: wave, wave + 8, ...  Their rows travel from global
// memory into the wave's own two half tiles in LDS (32 rows x 64 dimensions each, one read while the other lands; no barrier in
// the stream), while the tokens are operands in registers.  Per query the product is S^T = C Q^T, a lane owns one token; averaged
// it is S = Q C^T, a lane owns one cluster and the sum over the tokens runs in its registers.  Maximum and normaliser of a token
// are put together from the eight waves through LDS.
// Bound by its phases one after the other: 20 heads x 150 tokens x 613 clusters, by the workgroups' clocks: operands there 1.3 us,
// scores 3.5, maxima 1.9, normalisers 1.6; at 32 heads x 1024 tokens x 1024 clusters a workgroup's second block of tokens takes 9
// us, its first 16 (the centroids come from memory; without one XCD per head every XCD fetched all of them: 20).  Traced there:
// averaged 31.8 us against 20.5 + 21.6 of the two sliced passes, per query 47 with the attention's block table against 32.8 + 21.2,
// 59 with the tokens' key counts as well (the step 585 us on either path).  Counters there: matrix cores busy 13 % (averaged), no
// bank conflicts.  The form of four tiles per wave fills its 128 registers: the compiler puts 7 values (averaged 3) of the
// addresses and the start in scratch memory, 32 bytes a lane.
#include <algorithm>

#include "sq_common.hpp"
#include "sq_internal.hpp"
#include "sq_lookup.hpp"

namespace sq {

constexpr int LR_WAVES = 8, LR_THREADS = 64 * LR_WAVES;
constexpr int LR_BT = 32;                    // tokens per workgroup
constexpr int LR_HALF = 32 * 128;            // bytes of half a tile: 32 rows of 128 B

// TILES: tiles per wave, at most; two workgroups share a compute unit.
template <bool MEAN, int TILES>
__global__ __launch_bounds__(LR_THREADS, 4) void lookup_rows_kernel(
    const _Float16 *__restrict__ q, const _Float16 *__restrict__ cent, const int32_t *__restrict__ sizes,
    const float *__restrict__ thresh, uint32_t *__restrict__ keep_mask, int32_t *__restrict__ n_keys,
    float *__restrict__ part_sum, int n_part, int BH, int H, int Lq, int C, float sm_scale, BlockTable table)
{
    // Workgroups are dealt to the 8 XCDs round-robin by their id: those of a (sequence, head), which read the same centroids, are
    // made to land on one XCD.
    const int nbt = (Lq + LR_BT - 1) / LR_BT, n_blk = MEAN ? n_part : nbt, units = n_blk * BH;
    const int per_xcd = (units + 7) >> 3, extra = (int)blockIdx.x - 8 * per_xcd;
    if (!MEAN && extra >= 0) {                              // extra workgroups: the attention's block table
        const int groups = block_table_groups(table.nblk);
        block_table_part(table, extra / groups, extra % groups, LR_WAVES);
        return;
    }
    const int unit = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (unit >= units) return;
    constexpr int CMAX = TILES * LR_WAVES * 32;
    __shared__ __align__(16) unsigned char stage[LR_WAVES][2][LR_HALF];
    __shared__ __align__(16) float s_N[CMAX];               // cluster sizes as floats (exact: fewer than 2^24 keys a head)
    __shared__ __align__(16) float s_red[LR_WAVES][LR_BT];
    __shared__ __align__(16) float s_tok[2][LR_BT];         // MEAN: the tokens' largest scores, 1 / D
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5;
    const int bh = unit / n_blk, blk = unit - bh * n_blk, h = bh % H;
    const int nt = (C + 31) >> 5;                           // tiles
    const float c2 = sm_scale * 1.44269504088896341f;
    // Piece i of a half tile: rows i * 8 + lane / 8, 16-byte chunk (lane % 8) ^ (row / 2 % 8), so that the operand reads (16 rows
    // at one chunk index) fall into all banks.  Byte offset of this lane's part, in the first half.
    const uint32_t chunk = (uint32_t)((lane & 7) ^ (lane >> 4)) * 16u;
    auto row_at = [&](int t, int i) {
        int r = lane >> 3;
        asm volatile("" : "+v"(r));                         // (made where it is used, not kept for all tiles)
        return ((uint32_t)min((t * LR_WAVES + wave) * 32 + i * 8 + r, C - 1) * 256u + chunk) ^ (uint32_t)(i & 1) << 6;
    };
    for (int c = tid; c < nt * 32; c += LR_THREADS) s_N[c] = c < C ? (float)sizes[(size_t)h * C + c] : 0.0f;
    const char *ch = reinterpret_cast<const char *>(cent + (size_t)h * C * D);
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lk_lptr_t)&stage[wave][0][0]);
    auto fetch = [&](int t, int half) {                     // half tile -> its buffer, whose reads have come back
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_w + (uint32_t)(half * LR_HALF + i * 1024))),
                         "v"(row_at(t, i) + (uint32_t)half * 128u), "s"(ch) : "m0", "memory");
    };
    // (a barrier for what is in LDS: __syncthreads would wait for the tiles on their way as well)
    auto sync = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    const int mine = __builtin_amdgcn_readfirstlane(max(0, (nt - wave + LR_WAVES - 1) / LR_WAVES));   // this wave's tiles
    uint32_t rd[4];                                         // operand of step s of a half: row col, chunk 2 s + g
#pragma unroll
    for (int s = 0; s < 4; ++s) rd[s] = (uint32_t)(col * 128 + ((2 * s + g) ^ ((col >> 1) & 7)) * 16);
    const unsigned char *buf = &stage[wave][0][0];

    float csum[TILES];                                      // MEAN: this lane's cluster of every tile, summed over the tokens
#pragma unroll
    for (int t = 0; t < TILES; ++t) csum[t] = 0.0f;
    if (mine > 0) {
        fetch(0, 0);
        fetch(0, 1);
    }
    for (int tb = blk; tb < nbt; tb += n_blk) {
        const int t0 = tb * LR_BT;
        const bool again = MEAN && tb + n_part < nbt;       // the first tile is fetched again for the next tokens
        h8 bq[8];
        {
            const h8 *qp = reinterpret_cast<const h8 *>(q + ((size_t)bh * Lq + min(t0 + col, Lq - 1)) * D);
#pragma unroll
            for (int s = 0; s < 8; ++s) bq[s] = qp[s * 2 + g];
        }
        f16v x[TILES];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
#pragma unroll
            for (int r = 0; r < 16; ++r) x[t][r] = 0.0f;
            if (t >= mine) continue;                        // (wave-uniform)
            // the first half has landed when at most the second one's four loads are under way
            asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const h8 a = *reinterpret_cast<const h8 *>(buf + half * LR_HALF + rd[s]);
                    x[t] = MEAN ? __builtin_amdgcn_mfma_f32_32x32x16_f16(bq[4 * half + s], a, x[t], 0, 0, 0)
                                : __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bq[4 * half + s], x[t], 0, 0, 0);
                }
                if (t + 1 < mine) fetch(t + 1 < TILES ? t + 1 : 0, half);
                else if (again && mine > 1) fetch(0, half);  // (a wave's only tile is still there)
                else if (half == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (half == 0) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            }
        }
        if (tb == blk) sync();                              // s_N is there
        if constexpr (!MEAN) {
            // Lane: token col; rows 8 (r / 4) + 4 g + r % 4 of every tile.
            const float *Np = s_N + g * 4;
            auto n_of = [&](int t, float (&nv)[16]) {
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f4 v = *reinterpret_cast<const f4 *>(Np + (t * LR_WAVES + wave) * 32 + a * 8);
#pragma unroll
                    for (int k = 0; k < 4; ++k) nv[4 * a + k] = v[k];
                }
            };
            // A cluster without keys (or past the end) takes no part, whatever its centroid holds.
            float m = SQ_NEG_INF;
            uint32_t has[TILES];                            // the tile's clusters with keys
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                if (t >= mine) continue;
                has[t] = (uint32_t)__ballot(s_N[(t * LR_WAVES + wave) * 32 + col] > 0.0f);
                if (has[t] != ~0u) {                        // (uniform)
                    float nv[16];
                    n_of(t, nv);
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[t][r] = nv[r] > 0.0f ? x[t][r] : SQ_NEG_INF;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) m = fmaxf(m, x[t][r]);
            }
            m = cross32_max(m);
            if (g == 0) s_red[wave][col] = m;
            sync();
#pragma unroll
            for (int w = 0; w < LR_WAVES; ++w) m = fmaxf(m, s_red[w][col]);
            sync();                                // (s_red is used again)
            const float m_f = m == SQ_NEG_INF ? 0.0f : m;
            float sum = 0.0f;
            // (the difference first: it is exactly 0 for the largest score, so equal scores have equal, exact terms)
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                if (t >= mine) continue;
                float nv[16];
                n_of(t, nv);
#pragma unroll
                for (int r = 0; r < 16; ++r) sum = fmaf(nv[r], __builtin_amdgcn_exp2f((x[t][r] - m_f) * c2), sum);
            }
            sum = cross32_sum(sum);
            if (g == 0) s_red[wave][col] = sum;
            sync();
            float Dsum = 0.0f;
#pragma unroll
            for (int w = 0; w < LR_WAVES; ++w) Dsum += s_red[w][col];
            const float x_min = lk_least_kept(m, thresh[h] * Dsum, c2);
            const int W = (C + 31) >> 5;
            const size_t row = (size_t)bh * Lq + t0 + col;
            const bool valid = t0 + col < Lq;
            float keys = 0.0f;
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                if (t >= mine) continue;
                const int tile = t * LR_WAVES + wave;
                uint32_t bits = 0u;
#pragma unroll
                for (int r = 15; r >= 0; --r) {
                    uint32_t carry;
                    bits = __builtin_addc(bits, bits, (uint32_t)(x[t][r] >= x_min), &carry);
                }
                // bit 4 a + i -> bit 8 a + 4 g + i of the word; the other half of the wave holds the other bits
                bits = (bits | (bits << 8)) & 0x00ff00ffu;
                bits = (bits | (bits << 4)) & 0x0f0f0f0fu;
                const uint32_t word = cross32_or(bits << (4 * g)) & has[t];
                if (g == 0 && valid) keep_mask[row * W + tile] = word;
                if (n_keys)
                    for (int c = g; c < 32; c += 2) keys += (word >> c) & 1u ? s_N[tile * 32 + c] : 0.0f;
            }
            if (n_keys) {                                   // (uniform; exact in fp32, like the sizes)
                sync();
                keys = cross32_sum(keys);
                if (g == 0) s_red[wave][col] = keys;
                sync();
                if (tid < LR_BT && valid) {
                    float k = 0.0f;
                    for (int w = 0; w < LR_WAVES; ++w) k += s_red[w][col];
                    n_keys[row] = (int)k;
                }
            }
        } else {
            // Lane: cluster col of every tile; tokens 8 (r / 4) + 4 g + r % 4.
            float Nl[TILES];
#pragma unroll
            for (int t = 0; t < TILES; ++t) Nl[t] = t < mine ? s_N[(t * LR_WAVES + wave) * 32 + col] : 0.0f;
            // v[0..16) over the 32 lanes of each half wave: 16 -> 8 -> 4 -> 2 values per lane, each step combining what two
            // lanes (16, 1, 2 apart) hold and leaving either with half of the tokens, then the four lanes 4 apart.
            auto over_cols = [&](float (&v)[16], auto &&op) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {               // rows of 16 lanes: the even ones go on with tokens 0..7
                    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(v[r]), "+v"(v[r + 8]));
                    v[r] = op(v[r], v[r + 8]);
                }
                const bool odd1 = col & 1, odd2 = col & 2;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float keep = odd1 ? v[r + 4] : v[r], give = odd1 ? v[r] : v[r + 4];
                    v[r] = op(keep, dpp_f<0xb1>(give));
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const float keep = odd2 ? v[r + 2] : v[r], give = odd2 ? v[r] : v[r + 2];
                    v[r] = op(keep, dpp_f<0x4e>(give));
                    v[r] = op(v[r], dpp_f<0x128>(v[r]));
                    v[r] = op(v[r], dpp_f<0x124>(v[r]));
                }
            };
            auto fmx = [](float a, float b) { return fmaxf(a, b); };
            auto add = [](float a, float b) { return a + b; };
            // lane: values r = 0, 1 are index 8 (lane / 16 % 2) + 4 (lane % 2) + 2 (lane / 2 % 2) + r of its half's 16 tokens
            auto put = [&](const float (&v)[16]) {
                if ((col & 12) == 0) {
                    const int i = 8 * (col >> 4) + 4 * (col & 1) + (col & 2);
                    *reinterpret_cast<float2 *>(&s_red[wave][8 * (i >> 2) + 4 * g + (i & 3)]) = float2{v[0], v[1]};
                }
            };
            auto get = [&](const float *p, float (&v)[16]) {
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f4 u = *reinterpret_cast<const f4 *>(p + 8 * a + 4 * g);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[4 * a + k] = u[k];
                }
            };
            float v[16];
#pragma unroll
            for (int t = 0; t < TILES; ++t)
                if (__ballot(!(Nl[t] > 0.0f)) != 0ull)      // (uniform)
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[t][r] = Nl[t] > 0.0f ? x[t][r] : SQ_NEG_INF;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float m = x[0][r];
#pragma unroll
                for (int t = 1; t < TILES; ++t) m = fmaxf(m, x[t][r]);
                v[r] = m;
            }
            over_cols(v, fmx);
            put(v);
            sync();
            if (tid < LR_BT) {
                float m = s_red[0][tid];
#pragma unroll
                for (int w = 1; w < LR_WAVES; ++w) m = fmaxf(m, s_red[w][tid]);
                s_tok[0][tid] = m == SQ_NEG_INF ? 0.0f : m;
            }
            sync();
            get(s_tok[0], v);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float sum = 0.0f;
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    x[t][r] = __builtin_amdgcn_exp2f((x[t][r] - v[r]) * c2);
                    sum = fmaf(Nl[t], x[t][r], sum);
                }
                v[r] = sum;
            }
            over_cols(v, add);
            put(v);
            sync();
            if (tid < LR_BT) {
                float Dsum = 0.0f;
#pragma unroll
                for (int w = 0; w < LR_WAVES; ++w) Dsum += s_red[w][tid];
                s_tok[1][tid] = t0 + tid < Lq && Dsum > 0.0f ? 1.0f / Dsum : 0.0f;
            }
            sync();
            get(s_tok[1], v);
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) csum[t] = fmaf(x[t][r], v[r], csum[t]);
        }
    }
    if constexpr (MEAN) {
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int c = (t * LR_WAVES + wave) * 32 + col;
            const float s = cross32_sum(csum[t]);
            if (g == 0 && c < C) part_sum[((size_t)bh * n_part + blk) * C + c] = s_N[c] > 0.0f ? s : 0.0f;
        }
    }
}

// A row of 32 to 1024 clusters per 32 tokens is the work of one workgroup: long rows of few tokens and heads leave the chip idle
// and are scored in slices over two launches instead.  Whole steps, two launches (one, per query with
// 75 clusters) / this kernel, us, 32 keys per cluster:
//                              per query, clusters                            averaged, clusters
//                              75           500            1000               75           500            1000
//    1 head  x   16 tokens    22.0 / 19.8  31.9 / 28.5    37.9 / 37.2        22.1 / 20.7  25.1 / 23.2    29.7 / 30.0
//    8 heads x   47           23.9 / 20.9  40.3 / 36.9    53.5 / 55.0        24.7 / 21.4  34.8 / 34.2    37.2 / 38.9
//   16 heads x   64           27.2 / 23.7  53.0 / 50.2    81.3 / 80.9        25.1 / 22.8  35.7 / 34.9    43.8 / 45.5
//   20 heads x  150           35.0 / 31.5  80.8 / 74.9   128.0 / 121.3       31.2 / 27.6  39.8 / 36.5    70.9 / 68.8
//   24 heads x  333           44.2 / 41.5 115.4 / 106.9  193.7 / 186.2       37.0 / 34.8  55.4 / 50.8    70.2 / 67.3
//   32 heads x 1024           88.2 / 88.9 311.6 / 304.9  567.9 / 567.4       69.0 / 66.2 111.1 / 106.8  168.1 / 159.8
bool lookup_in_rows(int BH, int Lq, int C)
{
    return C <= LR_MAX_C && (C <= 2 * LR_WAVES * 32 || (long long)BH * ((Lq + LR_BT - 1) / LR_BT) >= 64);
}

// Averaged: parts the tokens are dealt to, two workgroups per compute unit.
int lookup_rows_parts(int BH, int Lq) { return std::clamp(512 / BH, 1, (Lq + LR_BT - 1) / LR_BT); }

hipError_t launch_lookup_rows(const void *q, const void *centroids, const int32_t *sizes, const float *thresh,
                              uint32_t *keep_mask, int32_t *n_keys, float *part_sum, bool mean, int B, int H, int Lq, int C,
                              float sm_scale, hipStream_t s, const BlockTable *table)
{
    if (C > LR_MAX_C || (table && mean)) return hipErrorInvalidValue;
    const int BH = B * H, nbt = (Lq + LR_BT - 1) / LR_BT, n_part = lookup_rows_parts(BH, Lq);
    const int units = (mean ? n_part : nbt) * BH, extra = table ? block_table_groups(table->nblk) * H : 0;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((units + 7) / 8 * 8 + extra), dim3(LR_THREADS), 0, s, (const _Float16 *)q,
                           (const _Float16 *)centroids, sizes, thresh, keep_mask, n_keys, part_sum, n_part, BH, H, Lq, C, sm_scale,
                           table ? *table : BlockTable{});
    };
    static_assert(LR_MAX_C == 4 * LR_WAVES * 32, "up to four tiles per wave");
    if (C <= LR_WAVES * 32) mean ? launch(lookup_rows_kernel<true, 1>) : launch(lookup_rows_kernel<false, 1>);
    else if (C <= 2 * LR_WAVES * 32) mean ? launch(lookup_rows_kernel<true, 2>) : launch(lookup_rows_kernel<false, 2>);
    else mean ? launch(lookup_rows_kernel<true, 4>) : launch(lookup_rows_kernel<false, 4>);
    return hipGetLastError();
}

}  // namespace sq
