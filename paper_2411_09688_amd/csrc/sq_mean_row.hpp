// A row's selection on averaged scores (Appendix D, "Prefill Stage") by a whole workgroup, for launches that make the kept set they
// walk by themselves: what mean_select_kernel does in a launch of its own.
#pragma once
#include "sq_common.hpp"
#include "sq_internal.hpp"
#include "sq_lookup.hpp"

namespace sq {

// Words of LDS for a row of at most MAX_C clusters: positions, first entries, the number of records, counts per group of 64.
// (Candidates: the mask behind them.)
constexpr int mean_row_words(int max_c) { return 2 * max_c + 1 + 2 * (max_c / 64); }
constexpr int mean_row_cand_words(int max_c) { return mean_row_words(max_c) + max_c / 32; }

// The entries a (sequence, head) emits: its kept clusters' keys or, with CHILDREN, the kept clusters' children one level down.  Parts
// of the clusters' averaged scores are added in ascending order, divided by the tokens and compared with the threshold
// (mean_select_kernel's decision).  Left in LDS: s[0..kept) positions of the emitting clusters' first entries in the row's list,
// s[MAX_C ..) those entries; s[2 MAX_C] the number of emitting clusters.  Returns the length of the list.  A barrier at the end.
// write: the mask and the count, too.  CANDS: the row's clusters are its candidates, sums in their order (see mean_select_kernel).
template <int WAVES, int MAX_C, bool CHILDREN, bool CANDS>
__device__ __forceinline__ int mean_row_select(const PfSelect &sel, size_t bh, int h, int C_all, int Lq, bool write, int *s)
{
    constexpr int THREADS = 64 * WAVES, STEPS = MAX_C / THREADS, GROUPS = MAX_C / 64;
    static_assert(GROUPS <= 64, "a group's counts per lane");
    int *s_pos = s, *s_first = s + MAX_C, *s_n = s_first + MAX_C, *s_cnt = s_n + 1, *s_len = s_cnt + GROUPS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), W = (C_all + 31) >> 5;
    const int C = CANDS ? min(sel.cand_hdr[bh].y, C_all) : C_all;   // entries
    const int parts = CANDS ? lookup_mean_parts(sel.rows, Lq, C) : sel.parts;
    const float *ps = sel.part_sum + (CANDS ? bh * lookup_cand_stride(sel.rows, C_all) : bh * parts * C);
    const int32_t *N = sel.sizes + (size_t)h * C_all, *off = sel.offsets + (size_t)h * (C_all + 1);
    const int32_t *cid = CANDS ? sel.cand_id + bh * C_all : nullptr;
    uint32_t *s_mask = reinterpret_cast<uint32_t *>(s + mean_row_words(MAX_C));   // CANDS
    if (CANDS)
        for (int w = tid; w < W; w += THREADS) s_mask[w] = 0u;
    const float T = sel.thresh[h], div = (float)Lq;
    if (tid < GROUPS) s_cnt[tid] = s_len[tid] = 0;
    int first[STEPS], len[STEPS], child[STEPS];             // (child: the end of the children)
    float sum[STEPS];
    int id[CANDS ? STEPS : 1];
    if constexpr (CANDS)
#pragma unroll
        for (int k = 0; k < STEPS; ++k) id[k] = k * THREADS < C ? min(max(cid[min(k * THREADS + tid, C - 1)], 0), C_all - 1) : 0;
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        const int i = CANDS ? id[CANDS ? k : 0] : min(k * THREADS + tid, C - 1);
        sum[k] = 0.0f;
        len[k] = first[k] = child[k] = 0;
        if (k * THREADS < C) {                              // (uniform)
            len[k] = N[i];
            first[k] = off[i];
            if (CHILDREN) child[k] = off[i + 1];
        }
    }
    constexpr int AHEAD = 8;                                // parts under way together
    for (int p0 = 0; p0 < parts; p0 += AHEAD)
#pragma unroll
        for (int k = 0; k < STEPS; ++k) {
            if (k * THREADS >= C) break;                    // (uniform)
            const float *at = ps + min(k * THREADS + tid, C - 1);
            float v[AHEAD];
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) v[p] = at[(size_t)min(p0 + p, parts - 1) * C];
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) sum[k] = p0 + p < parts ? sum[k] + v[p] : sum[k];
        }
    __syncthreads();                                        // (the counts are zero)
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        if (k * THREADS >= C) break;
        const bool keep = k * THREADS + tid < C && len[k] > 0 && sum[k] / div > T;
        len[k] = !keep ? 0 : CHILDREN ? max(child[k] - first[k], 0) : len[k];
        const unsigned long long bal = __ballot(keep), emit = __ballot(len[k] > 0);
        const int total = wave_sum_i(len[k]), g = k * WAVES + wave;
        if (CANDS && write && sel.keep_mask) wave_mask_or(s_mask, id[CANDS ? k : 0], keep, lane);
        if (lane == 0) {
            s_cnt[g] = __popcll(emit);
            s_len[g] = total;
            if (!CANDS && write && sel.keep_mask && 2 * g < W) {
                sel.keep_mask[bh * W + 2 * g] = (uint32_t)bal;
                if (2 * g + 1 < W) sel.keep_mask[bh * W + 2 * g + 1] = (uint32_t)(bal >> 32);
            }
        }
    }
    __syncthreads();
    const int gc = lane < GROUPS ? s_cnt[lane] : 0, gl = lane < GROUPS ? s_len[lane] : 0;
    const int ic = wave_inclusive_scan(gc, lane), il = wave_inclusive_scan(gl, lane);
    const int kept = __builtin_amdgcn_readlane(ic, 63), keys = __builtin_amdgcn_readlane(il, 63);
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        if (k * THREADS >= C) break;
        const int g = k * WAVES + wave;
        const unsigned long long bal = __ballot(len[k] > 0);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
        const int c = __builtin_amdgcn_readlane(ic - gc, g) + rank;
        const int pos = __builtin_amdgcn_readlane(il - gl, g) + wave_inclusive_scan(len[k], lane) - len[k];
        if (len[k] > 0) {
            s_pos[c] = pos;
            s_first[c] = first[k];
        }
    }
    if (tid == 0) {
        *s_n = kept;
        if (write && sel.n_keys) sel.n_keys[bh] = keys;
    }
    __syncthreads();
    if (CANDS && write && sel.keep_mask)
        for (int w = tid; w < W; w += THREADS) sel.keep_mask[bh * W + w] = s_mask[w];
    return keys;
}

}  // namespace sq
