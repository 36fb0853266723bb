// Centroid lookup for prefill (Section 4.1) without a [queries x clusters] intermediate in memory, in two launches that each
// stream the centroids once; both are spread over (sequence, head) x blocks of query tokens x slices of the clusters, so that
// a few tokens or heads still fill the chip.  (Rows whose scores fit the registers of a workgroup: sq_lookup_rows.hip.)
//
//   lookup_pass_kernel<LK_STATS>        per (token, slice): the largest score r and sum_i N_i exp(x_i - r) over the slice's
//                  clusters (Eq. 1's normaliser), 8 bytes each.
//   then, with the slices' pairs merged per token:
//   lookup_pass_kernel<LK_DECIDE>       per-query selection: keep cluster i for token t iff N_i > 0 and
//                  exp(x_i - m) > T * D, compared as x_i >= the least score that passes (lk_least_kept): one comparison per
//                  (token, cluster), its bit shifted into the token's mask word.
//   (lookup_pass_kernel<LK_BOTH>        both in one launch, for rows of few clusters with per-token candidates)
//   mean_scores_kernel                  selection on averaged scores (Appendix D, "Prefill Stage"), first half: the scores
//                  S_i(t) = exp(x_i - m) / D are summed over the tokens per cluster and written as part_sum
//                  [B*H, lookup_parts(), C]; mean_select_kernel adds the parts.
//   CANDS == true  (averaged scores) second level of a hierarchical lookup (Section 3.3, Eq. 3): the clusters scored are the
//                  n candidates cand_id[bh, 0..n) of the (sequence, head) -- the children of the coarse clusters kept
//                  one level up -- so the normaliser runs over the candidates only; part_sum is written in candidate order.
//   PARENTS == true (per-query selection) second level of a hierarchical lookup with per-token candidates: fine
//                  cluster i counts for token t only if t kept its parent coarse cluster (bit parent[i] of the
//                  token's level-1 mask); the others are treated like clusters without keys.
//
// Scores run on the matrix cores in 32x32x16 fp16 tiles.  In the passes a wave owns 32 tokens (S^T = C Q^T: a lane owns one
// token column and 16 clusters per tile, so normaliser and threshold test are per-lane scalars) and the four waves of a
// workgroup share the centroid stream, groups of 64 that travel straight from global memory into one of two LDS buffers.  The
// averaged form is turned round (S = Q C^T: a lane owns one cluster column and sums over the tokens in its registers; the
// waves share the staged queries).  Bound by vector instructions: 6 per (token, cluster) in the first pass, 3 in the second.
// 32 heads x 1024 tokens x 1024 clusters, traced: sums 20.9 us by themselves and 32.7 with the block table of the attention in the
// same launch, decisions 22, averages 22 (one launch of two passes over 16x16x32 tiles, a workgroup per 64 tokens and no block
// table in it: 55 us, averaged 61); 20 heads x 150 tokens x 613 clusters 6.8 + 6.1 against 26.
#include <algorithm>
#include <type_traits>

#include "sq_common.hpp"
#include "sq_internal.hpp"
#include "sq_lookup.hpp"
#include "sq_mean_row.hpp"

namespace sq {

constexpr int LK_G = 64;                     // centroids per staged group
constexpr int LK_BT = 128;                   // tokens per workgroup (four waves x 32)
// With per-token candidates, rows of at most so many clusters are decided in one launch.  Whole steps over two levels (16 coarse
// clusters, three tenths kept), two launches / one, us, 32 keys per cluster:
//   clusters                     75            128            192            250            320
//    1 head  x   16 tokens   31.3 / 28.8    31.5 / 29.8    32.0 / 33.2    31.8 / 36.2    32.1 / 40.4
//   16 heads x   28 tokens   35.3 / 34.0    38.5 / 37.4    37.9 / 39.8    38.5 / 44.3    39.5 / 48.6
//    4 heads x  333 tokens   43.3 / 42.6    46.7 / 45.8    47.5 / 49.5    47.6 / 53.9    50.0 / 58.9
//   32 heads x 1024 tokens    98.5 / 97.1  117.8 / 114.9  143.3 / 140.1  157.5 / 159.2  179.9 / 177.1
constexpr int LK_ONE_C = 128;
constexpr int LK_COARSE_MAX = 1024;          // coarse clusters that the pass over the candidates selects from
constexpr int LK_MAX_GROUPS = 32;            // groups of a slice's candidates that it holds, at most
constexpr int LK_MAX_W1 = 32;                // level-1 mask words per token held in LDS: at most 1024 coarse clusters

// A token's pairs (r, sum) of the slices first, first + STEP, ... (at most LK_MAX_SLICES / STEP of them): the loads are issued
// together and merged later, so that their latency lies under the work in between.
template <int STEP>
struct SlicePairs {
    float2 v[LK_MAX_SLICES / STEP];
    __device__ __forceinline__ void load(const float2 *st, int first, int n_slice)
    {
#pragma unroll
        for (int k = 0; k < LK_MAX_SLICES / STEP; ++k) {
            v[k] = float2{SQ_NEG_INF, 0.0f};
            if (k * STEP < n_slice) {                       // (uniform: one jump past the slices there are not)
                const int s = first + k * STEP;
                if (s < n_slice) v[k] = st[s];
            }
        }
    }
    __device__ __forceinline__ float largest() const
    {
        float m = SQ_NEG_INF;
#pragma unroll
        for (int k = 0; k < LK_MAX_SLICES / STEP; ++k) m = fmaxf(m, v[k].x);
        return m;
    }
    __device__ __forceinline__ float sum(float m, float c2) const   // relative to m >= largest(); 0 if nothing was scored
    {
        float d = 0.0f;
#pragma unroll
        for (int k = 0; k < LK_MAX_SLICES / STEP; ++k)
            if (v[k].y != 0.0f) d = fmaf(v[k].y, __builtin_amdgcn_exp2f((v[k].x - m) * c2), d);
        return d;
    }
};

// Which passes a launch makes.  BOTH: one launch for rows of few clusters, where a second launch costs more than slices give.
enum LkMode { LK_STATS, LK_DECIDE, LK_BOTH };

// CHILDREN (with CANDS, sums): the candidates are made here, from the parts of the coarse level's averaged scores (what
// mean_select_kernel does in a launch of its own otherwise); the first token block's workgroups write cand_id and cand_hdr for the
// launches behind.
template <LkMode MODE, bool CANDS, bool PARENTS, bool KEYS, bool CHILDREN>
__global__ __launch_bounds__(256) void lookup_pass_kernel(
    const _Float16 *__restrict__ q, const _Float16 *__restrict__ cent, const int32_t *__restrict__ sizes,
    const float *__restrict__ thresh, float2 *__restrict__ stats, uint32_t *__restrict__ keep_mask,
    int32_t *__restrict__ n_keys, const int32_t *cand_id, const int2 *cand_hdr,
    const uint32_t *__restrict__ mask1, int W1, int n_slice, int H, int Lq, int C_all, float sm_scale, BlockTable table,
    PfSelect coarse, int C1)
{
    if (MODE != LK_DECIDE && !CANDS) {                      // extra workgroups: the attention's block table
        const int extra = (int)blockIdx.x - (Lq + LK_BT - 1) / LK_BT * n_slice;
        if (extra >= 0) {
            if ((int)blockIdx.y < H) block_table_part(table, blockIdx.y, extra, 4);
            return;
        }
    }
    __shared__ __align__(16) unsigned char stage[2 * LK_G * D * 2];
    __shared__ __align__(16) float s_N[2][LK_G];            // cluster sizes as floats (exact: a head has fewer than 2^24 keys)
    __shared__ __align__(16) float s_start[2][LK_G];        // where a cluster's score products start: 0, or for a cluster
                                                            // without keys (or past the end) -inf -- it adds nothing -- or,
                                                            // when deciding, NaN: it passes no comparison
    __shared__ __align__(16) int s_par[2][PARENTS ? LK_G : 1];
    __shared__ uint32_t s_m1[PARENTS ? LK_BT * LK_MAX_W1 : 1];   // level-1 masks of the workgroup's tokens
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5, l16 = lane & 15;
    const int bh = blockIdx.y, h = bh % H, slice = blockIdx.x % n_slice;
    const int t0 = (int)(blockIdx.x / n_slice) * LK_BT;
    // C: the clusters scored (all of the head's, or the candidates); C_all: row length of the arrays.
    __shared__ int s_ids[CHILDREN ? LK_MAX_GROUPS * LK_G : 1];   // CHILDREN: the slice's candidates
    int n_cand = 0;
    if constexpr (CHILDREN) {
        static_assert(sizeof(stage) >= mean_row_words(LK_COARSE_MAX) * sizeof(int), "the records lie where the centroids will be");
        n_cand = mean_row_select<4, LK_COARSE_MAX, true, false>(coarse, bh, h, C1, Lq, false, reinterpret_cast<int *>(stage));
    } else if constexpr (CANDS)
        n_cand = cand_hdr[bh].y;
    const int C = CANDS ? min(n_cand, C_all) : C_all;
    const int ng = (C + LK_G - 1) / LK_G, per = (ng + n_slice - 1) / n_slice;
    const int g0 = min(slice * per, ng), g1 = min(g0 + per, ng);
    const int t = t0 + wave * 32 + col;                     // this lane's token (past the end: the last one, not stored)
    const bool valid = t < Lq;
    const size_t row = (size_t)bh * Lq + min(t, Lq - 1);
    const int W = (C + 31) >> 5;
    const float c2 = sm_scale * 1.44269504088896341f;       // base-2 exponents: one instruction per exponential
    const int32_t *cid = CANDS ? cand_id + (size_t)bh * C_all : nullptr;
    if constexpr (CHILDREN) {
        const int *s_pos = reinterpret_cast<const int *>(stage), *s_first = s_pos + LK_COARSE_MAX;
        const int emit = s_pos[2 * LK_COARSE_MAX], p0 = g0 * LK_G, p1 = min(g1 * LK_G, C);
        for (int p = p0 + tid; p < p1; p += 256) {
            int k = 0;                                      // the kept coarse cluster whose children p is one of
#pragma unroll
            for (int step = LK_COARSE_MAX / 2; step > 0; step >>= 1)
                if (k + step < emit && s_pos[k + step] <= p) k += step;
            const int id = min(max(s_first[k] + p - s_pos[k], 0), C_all - 1);
            s_ids[p - p0] = id;
            if (t0 == 0) const_cast<int32_t *>(cand_id)[(size_t)bh * C_all + p] = id;
        }
        if (t0 == 0 && slice == 0 && tid == 0) const_cast<int2 *>(cand_hdr)[bh] = int2{emit, n_cand};
        __syncthreads();                                    // (the records are read)
    }
    const int32_t *par = PARENTS ? cand_id + (size_t)h * C_all : nullptr;     // (PARENTS: cand_id is parent [H, C])
    if (KEYS && MODE == LK_STATS && slice == 0 && g == 0 && valid) n_keys[row] = 0;   // (summed over the slices by the second pass)
    if (MODE == LK_DECIDE && g0 >= g1) return;              // (workgroup-uniform)
    if (PARENTS)
        for (int idx = tid; idx < LK_BT * W1; idx += 256) {
            const int r = idx / W1, w = idx - r * W1;
            s_m1[r * W1 + w] = mask1[((size_t)bh * Lq + min(t0 + r, Lq - 1)) * W1 + w];
        }
    h8 bq[8];
    {
        const h8 *qp = reinterpret_cast<const h8 *>(q + row * D);
#pragma unroll
        for (int s = 0; s < 8; ++s) bq[s] = qp[s * 2 + g];
    }
    float x_min = 0.0f;                                     // the least raw score that is kept
    SlicePairs<MODE == LK_DECIDE ? 2 : LK_MAX_SLICES> sp;   // (the two lanes of a token take every other slice)
    if (MODE == LK_DECIDE) sp.load(stats + row * n_slice, g, n_slice);

    const char *ch = reinterpret_cast<const char *>(cent + (size_t)h * C_all * D);
    const int32_t *Nh = sizes + (size_t)h * C_all;
    const int trow = tid >> 4;
    const uint32_t chunk = (uint32_t)((tid & 15) ^ (trow & 15)) * 16u;
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lk_lptr_t)stage) + (uint32_t)wave * 1024u;
    int id_n[4] = {}, id_s = 0;                             // CANDS: rows of the group after next, and this thread's cluster of it
    auto cluster_at = [&](int c) {                          // (a group past the slice's last one is never used)
        if constexpr (CHILDREN) return s_ids[min(c, min(g1 * LK_G, C) - 1) - g0 * LK_G];
        else return CANDS ? min(max(cid[c], 0), C_all - 1) : c;
    };
    auto fetch_ids = [&](int gr) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = min(gr * LK_G + i * 16 + trow, C - 1);
            id_n[i] = cluster_at(c);
        }
        id_s = cluster_at(min(gr * LK_G + (tid & (LK_G - 1)), C - 1));
    };
    int pn = 0, pp = 0;
    auto fetch = [&](int gr, int buf) {                     // group gr -> buffer buf (its rows' ids are in id_n)
#pragma unroll
        for (int i = 0; i < 4; ++i) lk_stage(ch, (uint32_t)id_n[i] * 256u + chunk, lds_w + (uint32_t)(buf * (LK_G * 256) + i * 4096));
        if (tid < LK_G) {                                   // 0 past the last cluster
            const int c = gr * LK_G + tid;
            pn = c < C ? Nh[id_s] : 0;
            if (PARENTS) pp = c < C ? min(max(par[c], 0), W1 * 32 - 1) : 0;
        }
    };
    auto commit = [&](int buf, bool decide) {
        if (tid < LK_G) {
            s_N[buf][tid] = (float)pn;
            s_start[buf][tid] = pn > 0 ? 0.0f : decide ? __builtin_nanf("") : SQ_NEG_INF;
            if (PARENTS) s_par[buf][tid] = pp;
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);                 // this wave's loads to LDS have landed
    };

    float ref = SQ_NEG_INF, ref_f = 0.0f, Dsum = 0.0f, keys = 0.0f;   // largest score seen; the same, 0 before there is one
    auto sweep = [&](auto pass2) {
        constexpr bool DECIDE = decltype(pass2)::value;
        if (g0 < g1) {
            fetch_ids(g0);
            fetch(g0, 0);
            fetch_ids(g0 + 1);
            if (MODE == LK_DECIDE) {                        // (under the loads of the first group)
                const float m = cross32_max(sp.largest());
                x_min = lk_least_kept(m, thresh[h] * cross32_sum(m == SQ_NEG_INF ? 0.0f : sp.sum(m, c2)), c2);
            }
            commit(0, DECIDE);
        }
        __syncthreads();
        for (int gr = g0; gr < g1; ++gr) {
            const int buf = (gr - g0) & 1;
            if (gr + 1 < g1) {
                fetch(gr + 1, buf ^ 1);
                fetch_ids(gr + 2);
            }
            const _Float16 *tile = reinterpret_cast<const _Float16 *>(stage + buf * (LK_G * 256));
            uint32_t words[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f16v acc;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f4 v = *reinterpret_cast<const f4 *>(&s_start[buf][u * 32 + a * 8 + g * 4]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc[4 * a + k] = v[k];
                }
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const h8 a = *reinterpret_cast<const h8 *>(tile + (u * 32 + col) * D + ((2 * s + g) ^ l16) * 8);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bq[s], acc, 0, 0, 0);
                }
                float nv[16];
                if (!DECIDE || KEYS) {
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const f4 v = *reinterpret_cast<const f4 *>(&s_N[buf][u * 32 + a * 8 + g * 4]);
#pragma unroll
                        for (int k = 0; k < 4; ++k) nv[4 * a + k] = v[k];
                    }
                }
                if (PARENTS) {                                  // not a candidate of this lane's token: as if it had no keys
                    const uint32_t *mrow = s_m1 + (wave * 32 + col) * W1;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int p = s_par[buf][u * 32 + (r >> 2) * 8 + g * 4 + (r & 3)];
                        if (!((mrow[p >> 5] >> (p & 31)) & 1u)) {
                            if (!DECIDE || KEYS) nv[r] = 0.0f;
                            acc[r] = DECIDE ? __builtin_nanf("") : SQ_NEG_INF;
                        }
                    }
                }
                if (!DECIDE) {
                    float mx = SQ_NEG_INF;                  // (NaN if a score is)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = __builtin_elementwise_maximum(mx, acc[r]);
                    if (__ballot(!(mx <= ref)) != 0ull) {
                        if (__ballot(mx != mx) != 0ull) {
                            // a cluster without keys whose centroid is not finite has -inf + inf or NaN here: -inf again
                            mx = SQ_NEG_INF;
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                acc[r] = nv[r] > 0.0f ? acc[r] : SQ_NEG_INF;
                                mx = fmaxf(mx, acc[r]);
                            }
                        }
                        if (mx > ref) {
                            Dsum *= __builtin_amdgcn_exp2f((ref - mx) * c2);   // ref = -inf: Dsum is 0 and stays 0
                            ref = ref_f = mx;
                        }
                    }
                    // (the difference first: it is exactly 0 for the largest score, so equal scores have equal, exact terms)
#pragma unroll
                    for (int r = 0; r < 16; ++r) Dsum = fmaf(nv[r], __builtin_amdgcn_exp2f((acc[r] - ref_f) * c2), Dsum);
                } else {
                    uint32_t bits = 0u;
#pragma unroll
                    for (int r = 15; r >= 0; --r) {
                        uint32_t carry;
                        const uint32_t keep = acc[r] >= x_min;
                        bits = __builtin_addc(bits, bits, keep, &carry);
                        if (KEYS) keys += keep ? nv[r] : 0.0f;
                    }
                    // bit 4 a + i -> bit 8 a + 4 g + i of the word; the other half of the wave holds the other bits
                    bits = (bits | (bits << 8)) & 0x00ff00ffu;
                    bits = (bits | (bits << 4)) & 0x0f0f0f0fu;
                    words[u] = cross32_or(bits << (4 * g));
                }
            }
            if (DECIDE && g == 0 && valid) {
                keep_mask[row * W + 2 * gr] = words[0];
                if (2 * gr + 1 < W) keep_mask[row * W + 2 * gr + 1] = words[1];
            }
            if (gr + 1 < g1) commit(buf ^ 1, DECIDE);
            __syncthreads();
        }
    };
    if (MODE != LK_DECIDE) {
        sweep(std::false_type{});                           // the two halves of the wave hold the other clusters of the token
        const float mo = __shfl_xor(ref, 32), Do = __shfl_xor(Dsum, 32), M = fmaxf(ref, mo);
        const float wa = ref == SQ_NEG_INF ? 0.0f : __builtin_amdgcn_exp2f((ref - M) * c2);
        const float wb = mo == SQ_NEG_INF ? 0.0f : __builtin_amdgcn_exp2f((mo - M) * c2);
        Dsum = Dsum * wa + Do * wb;
        if (MODE == LK_BOTH) x_min = lk_least_kept(M, thresh[h] * Dsum, c2);
        else if (g == 0 && valid) stats[row * n_slice + slice] = float2{M, Dsum};
    }
    if (MODE != LK_STATS) {
        sweep(std::true_type{});
        const int k = KEYS ? (int)cross32_sum(keys) : 0;    // (exact in fp32, like the sizes)
        if (KEYS && g == 0 && valid) {
            if (MODE == LK_BOTH) n_keys[row] = k;
            else if (k) atomicAdd(&n_keys[row], k);
        }
    }
}

// CANDS: a row's workgroups are (part, block of clusters) of the parts its own number of candidates asks for.  Bound by the chain of
// a workgroup's tiles, one behind the other: 8 rows x 2000 of 16384 candidates x 512 tokens, traced, 17.6 us in the one part that
// 16384 clusters ask for (128 workgroups of eight tiles each), 10.2 in four; whole step 112.9 -> 104.9.
template <bool CANDS>
__global__ __launch_bounds__(256) void mean_scores_kernel(
    const _Float16 *__restrict__ q, const _Float16 *__restrict__ cent, const int32_t *__restrict__ sizes,
    const float2 *__restrict__ stats, float *__restrict__ part_sum, const int32_t *__restrict__ cand_id,
    const int2 *__restrict__ cand_hdr, int n_slice, int H, int Lq, int C_all, float sm_scale)
{
    __shared__ __align__(16) unsigned char stage[2 * LK_MT * D * 2];
    __shared__ __align__(16) float s_m[2][LK_MT], s_inv[2][LK_MT];   // per token: the largest score, 1 / D
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, g = lane >> 5, l16 = lane & 15;
    const int bh = blockIdx.z, h = bh % H;
    const int C = CANDS ? min(cand_hdr[bh].y, C_all) : C_all, blocks = (C + LK_MC - 1) / LK_MC;
    const int n_part = CANDS ? lookup_mean_parts(gridDim.z, Lq, C) : (int)gridDim.y;
    if (CANDS && (int)blockIdx.x >= blocks * n_part) return;   // (workgroup-uniform)
    const int part = CANDS ? (int)blockIdx.x / blocks : (int)blockIdx.y;
    const int c0 = (CANDS ? (int)blockIdx.x - part * blocks : (int)blockIdx.x) * LK_MC;
    float *sums = part_sum + (CANDS ? bh * lookup_cand_stride(gridDim.z, C_all) + (size_t)part * C
                                    : ((size_t)bh * n_part + part) * C_all);
    const float c2 = sm_scale * 1.44269504088896341f;
    const int c = c0 + wave * 32 + col, cc = min(c, C - 1);
    const int id = CANDS ? min(max(cand_id[(size_t)bh * C_all + cc], 0), C_all - 1) : cc;
    h8 bc[8];                                               // this lane's centroid, B operand of S = Q C^T
    {
        const h8 *cp = reinterpret_cast<const h8 *>(cent + ((size_t)h * C_all + id) * D);
#pragma unroll
        for (int s = 0; s < 8; ++s) bc[s] = cp[s * 2 + g];
    }
    const bool keys = sizes[(size_t)h * C_all + id] > 0;
    const int nt = (Lq + LK_MT - 1) / LK_MT;
    const char *qh = reinterpret_cast<const char *>(q + (size_t)bh * Lq * D);
    const int trow = tid >> 4;
    const uint32_t chunk = (uint32_t)((tid & 15) ^ (trow & 15)) * 16u;
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lk_lptr_t)stage) + (uint32_t)wave * 1024u;
    SlicePairs<4> sp;
    int st_t = 0;
    auto fetch = [&](int tile, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            lk_stage(qh + (size_t)tile * (LK_MT * 256), (uint32_t)min(i * 16 + trow, Lq - 1 - tile * LK_MT) * 256u + chunk,
                     lds_w + (uint32_t)(buf * (LK_MT * 256) + i * 4096));
        st_t = tile * LK_MT + (tid >> 2);
        sp.load(stats + ((size_t)bh * Lq + min(st_t, Lq - 1)) * n_slice, tid & 3, n_slice);
    };
    auto commit = [&](int buf) {
        float m = sp.largest();                             // the four lanes of a token take every fourth slice
        m = fmaxf(m, dpp_f<0xb1>(m));
        m = fmaxf(m, dpp_f<0x4e>(m));
        float Dsum = m == SQ_NEG_INF ? 0.0f : sp.sum(m, c2);
        Dsum += dpp_f<0xb1>(Dsum);
        Dsum += dpp_f<0x4e>(Dsum);
        if ((tid & 3) == 0) {
            s_m[buf][tid >> 2] = m == SQ_NEG_INF ? 0.0f : m;
            s_inv[buf][tid >> 2] = st_t < Lq && Dsum > 0.0f ? 1.0f / Dsum : 0.0f;
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);                 // this wave's loads to LDS have landed
    };
    float sum = 0.0f;
    if (part < nt) {
        fetch(part, 0);
        commit(0);
    }
    __syncthreads();
    int buf = 0;
    for (int tile = part; tile < nt; tile += n_part, buf ^= 1) {
        if (tile + n_part < nt) fetch(tile + n_part, buf ^ 1);
        const _Float16 *qt = reinterpret_cast<const _Float16 *>(stage + buf * (LK_MT * 256));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f16v acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const h8 a = *reinterpret_cast<const h8 *>(qt + (u * 32 + col) * D + ((2 * s + g) ^ l16) * 8);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bc[s], acc, 0, 0, 0);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f4 mv = *reinterpret_cast<const f4 *>(&s_m[buf][u * 32 + a * 8 + g * 4]);
                const f4 iv = *reinterpret_cast<const f4 *>(&s_inv[buf][u * 32 + a * 8 + g * 4]);
#pragma unroll
                for (int k = 0; k < 4; ++k) sum = fmaf(__builtin_amdgcn_exp2f((acc[4 * a + k] - mv[k]) * c2), iv[k], sum);
            }
        }
        if (tile + n_part < nt) commit(buf ^ 1);
        __syncthreads();
    }
    sum = cross32_sum(sum);
    if (g == 0 && c < C) sums[c] = keys ? sum : 0.0f;
}

// Slices of the clusters: about two workgroups per compute unit (32 heads x 1024 tokens x 1024 clusters, whole averaged step
// with 256 / 512 / 1024 / 2048 workgroups: 162 / 155 / 160 / 161 us; shapes that cannot fill the chip do not care).  Before
// there were slices the 8 heads x 512 tokens over 2000 of 16384 clusters ran on 64 workgroups: 144 us against 13 + 18.
int lookup_slices(int BH, int Lq, int C)
{
    const long long units = (long long)BH * ((Lq + LK_BT - 1) / LK_BT);
    const long long want = (512 + units - 1) / units, groups = (C + LK_G - 1) / LK_G;
    return (int)std::min({want, groups, (long long)LK_MAX_SLICES});
}

int lookup_parts(int BH, int Lq, int C)
{
    return lookup_in_rows(BH, Lq, C) ? lookup_rows_parts(BH, Lq) : lookup_mean_parts(BH, Lq, C);
}

// Parts * C * BH for this C and any smaller one, and BH * lookup_cand_stride().
size_t lookup_part_floats(int BH, int C)
{
    return std::max((size_t)BH * C + LK_MEAN_GROUPS * LK_MC, (size_t)std::max(BH, 512) * std::min(C, LR_MAX_C));
}

// The coarse selection inside the pass (about 2 us more of its prologue: a round of loads and three barriers) against a launch of its own
// (6.5 us, and the round trip to the list it leaves), whole two-level steps, us, own launch / inside, by heads x tokens x keys, fine /
// coarse clusters: 8 x 512 x 262144, 16384 / 256 99.0 / 94.6, 1 x 512 x 262144, 16384 / 256 57.7 / 52.7, 4 x 300 x 200000, 10000 / 100
// 68.2 / 63.5, 8 x 200 x 131072, 6000 / 64 69.9 / 64.8, 8 x 300 x 40000, 2000 / 40 56.7 / 52.3, 1 x 64 x 100000, 4000 / 64 38.4 / 32.4.
// Every further round of workgroups (three a compute unit) pays the 2 us again: 16 x 8192 x 32768, 2000 / 64 (1024 workgroups) 347.7 / 350.3,
// 32 x 4096 (1024) 348.1 / 351.1, 32 x 6000, 2000 / 1000 (1504) 506.9 / 510.5, 32 x 16384 x 16384, 1000 / 32 (4096) 822.6 / 827.2;
// 20 x 8192 x 40000, 1500 / 64 (1280) 494.2 / 490.7.
// The other line is what a slice holds in LDS: 8 KB of candidates beside 32 KB of centroids, three workgroups per compute unit.
bool lookup_selects_children(int BH, int Lq, int C, int C1)
{
    const int groups = (C + LK_G - 1) / LK_G, n_slice = lookup_slices(BH, Lq, C);
    return (long long)BH * ((Lq + LK_BT - 1) / LK_BT) * n_slice <= 3 * 256 && C1 <= LK_COARSE_MAX && (groups + n_slice - 1) / n_slice <= LK_MAX_GROUPS;
}

hipError_t launch_prefill_lookup(const void *q, const void *centroids, const int32_t *sizes, const float *thresh,
                                 float *stats, uint32_t *keep_mask, int32_t *n_keys, float *part_sum, bool mean,
                                 int B, int H, int Lq, int C, float sm_scale, hipStream_t s, const int32_t *cand_id,
                                 const int2 *cand_hdr, const int32_t *parent, const uint32_t *mask1, int C1,
                                 const BlockTable *table, const PfSelect *coarse)
{
    if (!parent && !cand_id && lookup_in_rows(B * H, Lq, C))
        return launch_lookup_rows(q, centroids, sizes, thresh, keep_mask, n_keys, part_sum, mean, B, H, Lq, C, sm_scale, s, table);
    const bool one = parent && C <= LK_ONE_C;
    const int BH = B * H, n_slice = one ? 1 : lookup_slices(BH, Lq, C);
    const dim3 grid((Lq + LK_BT - 1) / LK_BT * n_slice, BH);
    const _Float16 *qh = (const _Float16 *)q, *ch = (const _Float16 *)centroids;
    float2 *st = reinterpret_cast<float2 *>(stats);
    if (parent && (mean || cand_id || !mask1 || C1 <= 0 || (C1 + 31) / 32 > LK_MAX_W1)) return hipErrorInvalidValue;
    if ((cand_id && (!mean || !cand_hdr)) || (table && cand_id)) return hipErrorInvalidValue;
    if (coarse && (!cand_id || !lookup_selects_children(BH, Lq, C, C1))) return hipErrorInvalidValue;
    const int32_t *ids = parent ? parent : cand_id;
    const int W1 = (C1 + 31) / 32;
    auto pass = [&](auto mode, auto cands, auto parents, auto keys, auto children) {
        const dim3 all(grid.x + (mode != LK_DECIDE && table ? block_table_groups(table->nblk) : 0), grid.y);
        hipLaunchKernelGGL((lookup_pass_kernel<mode, cands, parents, keys, children>), all, dim3(256), 0, s, qh, ch, sizes, thresh, st,
                           keep_mask, n_keys, ids, cand_hdr, mask1, W1, n_slice, H, Lq, C, sm_scale,
                           table ? *table : BlockTable{}, coarse ? *coarse : PfSelect{}, C1);
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr std::integral_constant<LkMode, LK_STATS> first{};
    constexpr std::integral_constant<LkMode, LK_DECIDE> second{};
    constexpr std::integral_constant<LkMode, LK_BOTH> both{};
    if (mean) {
        const int blocks = (C + LK_MC - 1) / LK_MC;
        if (cand_id) {
            coarse ? pass(first, yes, no, no, yes) : pass(first, yes, no, no, no);
            const dim3 mgrid(std::max(blocks, LK_MEAN_GROUPS / BH), 1, BH);
            hipLaunchKernelGGL(mean_scores_kernel<true>, mgrid, dim3(256), 0, s, qh, ch, sizes, st, part_sum, ids, cand_hdr,
                               n_slice, H, Lq, C, sm_scale);
        } else {
            pass(first, no, no, no, no);
            const dim3 mgrid(blocks, lookup_mean_parts(BH, Lq, C), BH);
            hipLaunchKernelGGL(mean_scores_kernel<false>, mgrid, dim3(256), 0, s, qh, ch, sizes, st, part_sum, ids, cand_hdr,
                               n_slice, H, Lq, C, sm_scale);
        }
    } else {
        auto select = [&](auto parents, auto keys) {
            if constexpr (parents)
                if (one) return pass(both, no, parents, keys, no);
            pass(first, no, parents, keys, no);
            pass(second, no, parents, keys, no);
        };
        if (parent && n_keys) select(yes, yes);
        else if (parent) select(yes, no);
        else if (n_keys) select(no, yes);
        else select(no, no);
    }
    return hipGetLastError();
}

// parent[h, c] = the coarse cluster whose child range child_offsets[j] .. child_offsets[j+1]-1 holds fine cluster c
// (binary search; C1 - 1 for ids past the last range).
__global__ __launch_bounds__(256) void child_parent_kernel(const int32_t *__restrict__ child_offsets,
                                                           int32_t *__restrict__ parent, int C1, int C2)
{
    const int h = blockIdx.y, c = blockIdx.x * 256 + threadIdx.x;
    if (c >= C2) return;
    const int32_t *co = child_offsets + (size_t)h * (C1 + 1);
    int lo = 0, hi = C1;                                     // invariant: co[lo] <= c (co[0] = 0), answer in [lo, hi)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (co[mid] <= c) lo = mid;
        else hi = mid;
    }
    parent[(size_t)h * C2 + c] = lo;
}

hipError_t launch_child_parent(const int32_t *child_offsets, int32_t *parent, int H, int C1, int C2, hipStream_t s)
{
    hipLaunchKernelGGL(child_parent_kernel, dim3((C2 + 255) / 256, H), dim3(256), 0, s, child_offsets, parent, C1, C2);
    return hipGetLastError();
}

}  // namespace sq
