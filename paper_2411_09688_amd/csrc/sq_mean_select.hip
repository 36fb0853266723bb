// Selection on averaged scores (Appendix D, "Prefill Stage") straight into the list the next launch walks: from the partial
// score sums of the lookup to the row's list of kept keys (the key-index tensor of Section 4.2), or of candidate clusters where
// the kept clusters are coarse ones.  (Where prefill_selects() the attention launch does this by itself, where
// lookup_selects_children() the pass over the candidates.)
//
// One workgroup per ((sequence, head) row, slice of the row's clusters).  A workgroup adds up the averages of every cluster up
// to the end of its slice, so it knows without talking to the others how many keys are kept in front of its own; it writes its
// slice's mask words and list entries, and the last slice the row's counts.  Bound by a chain of two reads and two barriers.
// Traced against one workgroup per row that left records behind and a launch that expanded them: 32 rows x 1024 clusters
// 5.6 us against 5.7 + 5.4, 20 x 613 5.6 against 5.1 + 2.8, 8 rows x 2000 of 16384 candidates 7.1 against 13.2 + 5; whole steps
// 155.0 -> 152.8, 41.8 -> 39.9 and (both levels) 123.1 -> 112.3, two heads over 175 K keys in 7932 clusters 60.1 -> 50.7.
#include <algorithm>

#include "sq_common.hpp"
#include "sq_internal.hpp"
#include "sq_key_list.hpp"
#include "sq_lookup.hpp"

namespace sq {

constexpr int MS_THREADS = 1024, MS_WAVES = MS_THREADS / 64;
constexpr int MS_STEPS = SELECT_MAX_C / MS_THREADS;          // entries per thread, at most
constexpr int MS_GROUPS = SELECT_MAX_C / 64;                 // an entry group: one wave in one step
constexpr int MS_SLICE_GROUPS = 16;                          // of a slice, at most: its kept clusters lie in LDS

// CAND: the row's entries are its candidates cand_id[row, 0 .. cand_hdr[row].y), part_sum is in candidate order (row_parts not
// used, see lookup_mean_parts) and mask bits are set by cluster id.  children: a kept cluster stands for the offsets[i] .. offsets[i + 1] - 1 of the next level (a kept
// cluster without children emits nothing) instead of its N_i keys.  list [rows, list_len]; hdr[row] = (entries kept, length).
template <bool CAND, int MS_AHEAD>                           // MS_AHEAD: steps whose loads are in flight together
__global__ __launch_bounds__(MS_THREADS) void mean_select_kernel(
    const float *__restrict__ part_sum, int row_parts, int Lq, const float *__restrict__ thresh,
    const int32_t *__restrict__ sizes, const int32_t *__restrict__ offsets, const int32_t *__restrict__ cand_id,
    const int2 *__restrict__ cand_hdr, bool children, uint32_t *__restrict__ keep_mask, int32_t *__restrict__ n_keys,
    int2 *__restrict__ hdr, int32_t *__restrict__ list, int list_len, int nsl, int H, int C)
{
    __shared__ int s_cnt[MS_GROUPS], s_len[MS_GROUPS];       // per entry group: clusters that emit, what they emit
    __shared__ int4 s_rec[MS_SLICE_GROUPS * 64];
    __shared__ uint32_t s_mask[CAND ? SELECT_MAX_C / 32 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = (int)blockIdx.x / nsl, sl = (int)blockIdx.x - row * nsl, h = row % H;
    const int W = (C + 31) >> 5;
    const int n = CAND ? min(cand_hdr[row].y, C) : C, ng = (n + 63) >> 6;
    const int per = max(1, (ng + nsl - 1) / nsl);
    const int ga = sl * per, gb = min(ga + per, ng);         // this slice's groups
    if (ga >= ng && sl > 0) return;                          // (workgroup-uniform)
    const bool last = gb == ng;
    const int parts = CAND ? lookup_mean_parts((int)gridDim.x / nsl, Lq, n) : row_parts;
    const int part_len = CAND ? n : C;
    const float *ps = part_sum + (CAND ? row * lookup_cand_stride((int)gridDim.x / nsl, C) : (size_t)row * parts * C);
    const float div = (float)Lq;
    const int32_t *N = sizes + (size_t)h * C, *off = offsets + (size_t)h * (C + 1);
    const int32_t *cid = CAND ? cand_id + (size_t)row * C : nullptr;
    const float T = thresh[h];
    if (CAND && last && keep_mask) {
        for (int w = tid; w < W; w += MS_THREADS) s_mask[w] = 0u;
        __syncthreads();
    }
    int start[MS_STEPS], len[MS_STEPS];                      // of a kept cluster (len 0: nothing emitted)
    const int n_end = min(n, gb * 64);
#pragma unroll
    for (int st0 = 0; st0 < MS_STEPS; st0 += MS_AHEAD) {
        if (st0 * MS_THREADS >= n_end) break;                // (workgroup-uniform)
        int id[MS_AHEAD], Ni[MS_AHEAD], o0[MS_AHEAD], o1[MS_AHEAD];
        float sum[MS_AHEAD];
#pragma unroll
        for (int k = 0; k < MS_AHEAD; ++k) {
            const int i = min((st0 + k) * MS_THREADS + tid, n_end - 1);
            id[k] = CAND ? min(max(cid[i], 0), C - 1) : i;
            sum[k] = 0.0f;
        }
#pragma unroll
        for (int k = 0; k < MS_AHEAD; ++k) {
            Ni[k] = N[id[k]];
            o0[k] = off[id[k]];
            o1[k] = children ? off[id[k] + 1] : 0;
        }
        const float *at = ps + min(st0 * MS_THREADS + tid, n_end - 1);
#pragma unroll 4
        for (int p = 0; p < parts; ++p) {                    // parts added in ascending order
#pragma unroll
            for (int k = 0; k < MS_AHEAD; ++k)
                sum[k] += at[(size_t)p * part_len + (MS_AHEAD == 1 ? 0 : min(k * MS_THREADS, max(n_end - 1 - st0 * MS_THREADS - tid, 0)))];
        }
#pragma unroll
        for (int k = 0; k < MS_AHEAD; ++k) {
            const int st = st0 + k, g = st * MS_WAVES + wave;
            const bool keep = st * MS_THREADS + tid < n_end && Ni[k] > 0 && sum[k] / div > T;
            start[st] = o0[k];
            len[st] = keep ? max(0, children ? o1[k] - o0[k] : Ni[k]) : 0;
            const unsigned long long bal = __ballot(keep), emit = __ballot(len[st] > 0);
            const int total = wave_sum_i(len[st]);
            if (lane == 0 && g < gb) {
                s_cnt[g] = __popcll(emit);
                s_len[g] = total;
                if (!CAND && keep_mask && g >= ga) {
                    keep_mask[(size_t)row * W + 2 * g] = (uint32_t)bal;
                    if (2 * g + 1 < W) keep_mask[(size_t)row * W + 2 * g + 1] = (uint32_t)(bal >> 32);
                }
            }
            if (CAND && last && keep_mask && g < gb) wave_mask_or(s_mask, id[k], keep, lane);
        }
    }
    __syncthreads();
    // Counts in front of every group: lane l holds the exclusive prefixes of groups 4 l .. 4 l + 3 (every wave the same).
    int pc[5], pl[5];
    pc[0] = pl[0] = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int g = 4 * lane + k;
        pc[k + 1] = pc[k] + (g < gb ? s_cnt[g] : 0);
        pl[k + 1] = pl[k] + (g < gb ? s_len[g] : 0);
    }
    static_assert(MS_GROUPS == 256, "four groups per lane");
    const int before_c = wave_inclusive_scan(pc[4], lane) - pc[4], before_l = wave_inclusive_scan(pl[4], lane) - pl[4];
    auto at = [&](const int (&p)[5], int before, int g) {    // (g wave-uniform)
        const int k = g & 3, v = before + (k == 0 ? p[0] : k == 1 ? p[1] : k == 2 ? p[2] : p[3]);
        return __builtin_amdgcn_readlane(v, g >> 2);
    };
    const int all_c = __builtin_amdgcn_readlane(before_c + pc[4], 63), all_l = __builtin_amdgcn_readlane(before_l + pl[4], 63);
    const int first = ga < MS_GROUPS ? at(pc, before_c, ga) : 0;
#pragma unroll
    for (int st = 0; st < MS_STEPS; ++st) {
        const int g = __builtin_amdgcn_readfirstlane(st * MS_WAVES + wave);
        if (g >= ga && g < gb) {
            const int c0 = at(pc, before_c, g) - first, l0 = at(pl, before_l, g);
            const unsigned long long emit = __ballot(len[st] > 0);
            const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(emit >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)emit, 0));
            const int incl = wave_inclusive_scan(len[st], lane);
            if (len[st] > 0) s_rec[c0 + rank] = make_int4(start[st], len[st], l0 + incl - len[st], 0);
        }
    }
    if (last && tid == 0) {
        hdr[row] = make_int2(all_c, all_l);
        if (n_keys) n_keys[row] = all_l;
    }
    __syncthreads();
    if (CAND && last && keep_mask)
        for (int w = tid; w < W; w += MS_THREADS) keep_mask[(size_t)row * W + w] = s_mask[w];
    write_key_index(s_rec, all_c - first, list + (size_t)row * list_len, list_len, MS_THREADS);
}

hipError_t launch_mean_select(const float *part_sum, int parts, int Lq, const float *thresh, const int32_t *sizes,
                              const int32_t *offsets, const int32_t *cand_id, const int2 *cand_hdr, bool children,
                              uint32_t *keep_mask, int32_t *n_keys, int2 *hdr, int32_t *list, int list_len, int rows, int H,
                              int C, hipStream_t s)
{
    if (C > SELECT_MAX_C || (cand_id != nullptr) != (cand_hdr != nullptr)) return hipErrorInvalidValue;
    // A workgroup per compute unit; a slice holds 64 to 1024 clusters.  (Two, with more of the row added up again by every one:
    // 9.3 instead of 5.6 us at 32 rows x 1024 clusters, 10.1 instead of 7.1 at 8 rows x 2000 of 16384; half of one: the same.)
    const int groups = (C + 63) / 64, least = (groups + MS_SLICE_GROUPS - 1) / MS_SLICE_GROUPS;
    const int nsl = std::clamp(256 / rows, least, groups);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(rows * nsl), dim3(MS_THREADS), 0, s, part_sum, parts, Lq, thresh, sizes, offsets,
                           cand_id, cand_hdr, children, keep_mask, n_keys, hdr, list, list_len, nsl, H, C);
    };
    if (cand_id) C <= MS_THREADS ? launch(mean_select_kernel<true, 1>) : launch(mean_select_kernel<true, 4>);
    else C <= MS_THREADS ? launch(mean_select_kernel<false, 1>) : launch(mean_select_kernel<false, 4>);
    return hipGetLastError();
}

}  // namespace sq
