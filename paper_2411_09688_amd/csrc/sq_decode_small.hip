// Decode step of small rows in two launches (Sections 3.2, 4.1, 4.2; Appendix D "Generation Stage").
//
// A call over a short context is bound by its launches and by the round trips of the chain scores -> selection ->
// key-index list -> attention -> merge, not by bytes: the four launches of the key-index step take 14.9 us of GPU time
// (and 10.8 us of the calling thread) for 4 heads x 4096 keys x 64 clusters, keep 1/4, whose K/V rows are 0.5 us of HBM.
// Up to DS_MAX_C clusters the lookup of a row is a few KB of centroids, so every workgroup of a row repeats it instead
// of waiting for another launch to publish it; the same call takes 8.3 us, 8.1 of them without the attention: what is
// left is the chain of dependent reads of one workgroup and one launch boundary.
//
//   decode_small_kernel        `splits` workgroups per query row.  Each scores the row's clusters on the matrix cores (the
//                              tile and the order of the k-steps are score_kernel's: bit-identical logits), takes the
//                              keep decisions in the library's summation order, lists its own equal share of the row's
//                              kept keys followed by its user keys in LDS, and streams those rows.  Workgroup 0 of a row
//                              also writes the row's keep mask and key count.
//   decode_small_merge_kernel  folds the row's partial results.
#include <algorithm>

#include "sq_merge.hpp"
#include "sq_internal.hpp"

namespace sq {

constexpr int DS_TILES = DS_MAX_C / 64;          // 16-cluster score tiles per wave
constexpr int DS_BATCH = 64;                     // keys of one batch of loads: 16 per wave, 16 lanes per key row
static_assert(DS_MAX_C == 256, "one thread per cluster");

__global__ __launch_bounds__(256) void decode_small_kernel(
    const _Float16 *__restrict__ q, const _Float16 *__restrict__ cent, const int32_t *__restrict__ sizes,
    const int32_t *__restrict__ offsets, const float *__restrict__ thresh, const _Float16 *__restrict__ Kf,
    const _Float16 *__restrict__ Vf, const _Float16 *__restrict__ Ku, const _Float16 *__restrict__ Vu,
    uint32_t *__restrict__ keep_mask, int32_t *__restrict__ n_keys, float *__restrict__ partials, int rows, int H, int G,
    int L, int C, int U, int splits, float sm_scale)
{
    __shared__ float s_x[DS_MAX_C];
    __shared__ int s_pos[DS_MAX_C], s_start[DS_MAX_C];       // kept clusters: keys kept before it, its first key
    __shared__ float s_m[4], s_d[4];
    __shared__ int s_cnt[4], s_keys[4];
    __shared__ int s_key[DS_MAX_SHARE];                      // this workgroup's keys: fixed-context row, or ~(user key)
    __shared__ float s_part[4][PART_STRIDE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p = lane & 15, g = lane >> 4;
    const int row = (int)blockIdx.x % rows, part = (int)blockIdx.x / rows;
    const int h = (row / G) % H;

    // ---- scores: wave w takes the 16-cluster tiles w, w + 4, ...; the query is column 0 of the tile ----
    const h8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    const h8 *qp = reinterpret_cast<const h8 *>(q + (size_t)row * D);
    const h8 qv = qp[p];                                     // the attention's share of the query
    const int32_t n_i = tid < C ? sizes[(size_t)h * C + tid] : 0;
    const int32_t start_i = tid < C ? offsets[(size_t)h * (C + 1) + tid] : 0;
    const float T = thresh[h];
    h8 bq[4], a[DS_TILES][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) bq[s] = qp[s * 4 + g];
#pragma unroll
    for (int t = 0; t < DS_TILES; ++t) {
        const int i0 = (t * 4 + wave) * 16;
        if (i0 < C) {                                        // wave-uniform
            const h8 *cp = reinterpret_cast<const h8 *>(cent + ((size_t)h * C + min(i0 + p, C - 1)) * D);
#pragma unroll
            for (int s = 0; s < 4; ++s) a[t][s] = cp[s * 4 + g];
        }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) bq[s] = p == 0 ? bq[s] : zero8;
#pragma unroll
    for (int t = 0; t < DS_TILES; ++t) {
        const int i0 = (t * 4 + wave) * 16;
        if (i0 < C) {
            f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t][s], bq[s], acc, 0, 0, 0);
            if (p == 0) *reinterpret_cast<f4 *>(&s_x[i0 + g * 4]) = acc * sm_scale;
        }
    }
    __syncthreads();

    // ---- (m, D) of Eq. 1 and the keep decisions, thread v = cluster v: the library's one summation order ----
    const float x = s_x[tid];                                // (past C: not looked at, n_i is 0)
    float m = wave_max(n_i > 0 ? x : SQ_NEG_INF);
    if (lane == 0) s_m[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
    const float e = n_i > 0 ? expf(x - m) : 0.0f;
    const float d_w = wave_sum(n_i > 0 ? __fmaf_rn((float)n_i, e, 0.0f) : 0.0f);
    if (lane == 0) s_d[wave] = d_w;
    __syncthreads();
    float Dsum = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) Dsum += s_d[w];
    const bool keep = n_i > 0 && e > T * Dsum;
    const unsigned long long bal = __ballot(keep);
    const int kv = keep ? n_i : 0;
    const int incl = wave_inclusive_scan(kv, lane);
    if (lane == 63) {
        s_cnt[wave] = __popcll(bal);
        s_keys[wave] = incl;
    }
    if (keep_mask && part == 0 && lane == 0) {
        const int W = (C + 31) >> 5, w0 = wave * 2;
        if (w0 < W) keep_mask[(size_t)row * W + w0] = (uint32_t)bal;
        if (w0 + 1 < W) keep_mask[(size_t)row * W + w0 + 1] = (uint32_t)(bal >> 32);
    }
    __syncthreads();
    int c_base = 0, k_base = 0, n_c = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w == wave) {
            c_base = n_c;
            k_base = tot;
        }
        n_c += s_cnt[w];
        tot += s_keys[w];
    }
    if (keep) {
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
        s_pos[c_base + rank] = k_base + incl - kv;
        s_start[c_base + rank] = start_i;
    }
    if (n_keys && part == 0 && tid == 0) n_keys[row] = tot;
    // This workgroup's share of the row's keys: kept keys in ascending order (sizes that exceed the context stay inside
    // the tensor), then the user keys.
    const int fixed = max(0, min(tot, L)), total = fixed + U;
    const int share = max(DS_MIN_SHARE, (total + splits - 1) / splits);
    const int lo = min(total, part * share), n = __builtin_amdgcn_readfirstlane(min(total, lo + share) - lo);
    __syncthreads();
    for (int t = tid; t < n; t += 256) {
        const int pos = lo + t;
        int key = ~(pos - fixed);
        if (pos < fixed) {                                   // the last kept cluster that begins at or before pos
            int c = 0;
#pragma unroll
            for (int step = DS_MAX_C / 2; step > 0; step >>= 1)
                if (c + step < n_c && s_pos[c + step] <= pos) c += step;
            key = max(0, min(s_start[c] + pos - s_pos[c], L - 1));   // malformed offsets stay in the tensor
        }
        s_key[t] = key;
    }
    __syncthreads();

    // ---- attention over the share (plain loads: a short context stays in the caches from step to step; with
    // non-temporal ones 32 heads x 4096 keys take 15.0 us instead of 14.2): lane group g of wave w takes keys w * 4 + g + 16 i of a batch ----
    const _Float16 *Kh = Kf + (size_t)h * L * D + p * 8, *Vh = Vf + (size_t)h * L * D + p * 8;
    const _Float16 *Kr = Ku + (size_t)(row / G) * U * D + p * 8, *Vr = Vu + (size_t)(row / G) * U * D + p * 8;
    const int slot = wave * 4 + g;
    float m_run = SQ_NEG_INF, l_run = 0.0f, o[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = 0.0f;
    auto load = [&](int base, h8 (&kr)[4], h8 (&vr)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (base + i * 16 < n) {                         // uniform: a round without keys reads nothing
                const int key = s_key[min(base + i * 16 + slot, n - 1)];
                const bool fx = key >= 0;
                const size_t off = (size_t)(fx ? key : ~key) * D;
                kr[i] = *reinterpret_cast<const h8 *>((fx ? Kh : Kr) + off);
                vr[i] = *reinterpret_cast<const h8 *>((fx ? Vh : Vr) + off);
            } else {
                kr[i] = zero8;
                vr[i] = zero8;
            }
    };
    auto consume = [&](int base, const h8 (&kr)[4], const h8 (&vr)[4]) __attribute__((always_inline)) {
        float s[4], m_b = SQ_NEG_INF;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float d = row16_sum(dot8(qv, kr[i], 0.0f)) * sm_scale;
            s[i] = base + i * 16 + slot < n ? d : SQ_NEG_INF;
            m_b = fmaxf(m_b, s[i]);
        }
        const float m_n = fmaxf(m_run, cross16_max(m_b));
        const float sc = m_run == SQ_NEG_INF ? 0.0f : __expf(m_run - m_n);
        l_run *= sc;
#pragma unroll
        for (int u = 0; u < 8; ++u) o[u] *= sc;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float pr = s[i] == SQ_NEG_INF ? 0.0f : __expf(s[i] - m_n);
            l_run += pr;
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] += pr * (float)vr[i][u];
        }
        m_run = m_n;
    };
    h8 k0[4], v0[4], k1[4], v1[4];
    if (n > 0) load(0, k0, v0);
    for (int b = 0; b < n; b += 2 * DS_BATCH) {              // one batch computed while the next one streams in
        if (b + DS_BATCH < n) load(b + DS_BATCH, k1, v1);
        consume(b, k0, v0);
        if (b + DS_BATCH >= n) break;
        if (b + 2 * DS_BATCH < n) load(b + 2 * DS_BATCH, k0, v0);
        consume(b + DS_BATCH, k1, v1);
    }
    // ---- the four lane groups, then the four waves: one partial result (an empty share: m = -inf, o not written) ----
    const float l_w = cross16_sum(l_run);
    float ow[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) ow[u] = cross16_sum(o[u]);
    if (g == 0) {
        if (p == 0) {
            s_part[wave][0] = m_run;
            s_part[wave][1] = l_w;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s_part[wave][4 + p * 8 + u] = ow[u];
    }
    __syncthreads();
    if (tid < D) {
        const float M = fmaxf(fmaxf(s_part[0][0], s_part[1][0]), fmaxf(s_part[2][0], s_part[3][0]));
        float lsum = 0.0f, acc = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = s_part[w][0];
            const float sc = mw == SQ_NEG_INF ? 0.0f : __expf(mw - M);
            lsum += sc * s_part[w][1];
            acc += sc * s_part[w][4 + tid];
        }
        float *dst = partials + ((size_t)row * splits + part) * PART_STRIDE;
        if (tid == 0) {
            dst[0] = M;
            dst[1] = lsum;
        }
        if (n > 0) dst[4 + tid] = acc;
    }
}

__global__ __launch_bounds__(MERGE_THREADS) void decode_small_merge_kernel(const float *__restrict__ partials,
                                                                           _Float16 *__restrict__ out,
                                                                           float *__restrict__ lse, int splits)
{
    __shared__ float s_red[MERGE_GROUPS * 130];
    const int row = blockIdx.x;
    const float *mine = partials + (size_t)row * splits * PART_STRIDE;
    merge_row<true>([&](int c) { return mine + (size_t)c * PART_STRIDE; }, splits, out + (size_t)row * D,
                    lse ? lse + row : nullptr, s_red, threadIdx.x);
}

// Which calls are small, and into how many shares a row is cut.  The workgroups of a call are about two per compute unit:
// with one, the heavy rows of a call of uneven rows take longer (32 heads x 4096 keys: 15.0 us with two, 18.4 with one).
// A row's share counts every key of the row, kept or not, as the counts of the other rows are not known here: where
// shares are long, the workgroups of a row that keeps much hold the call up, and the key-index step, which cuts all rows'
// kept keys into equal shares, is the better one.  GPU time of the whole step, key-index / small, us:
//   share  64:  4 heads x  4096 keys,  64 clusters, keep 1/4   14.9 /  8.3
//   share 258:  2 heads x 16384 keys, 256 clusters, keep 1/4   15.8 / 10.2
//   share 260: 16 heads x  8192 keys, 256 clusters, keep 1/8   17.1 / 16.0
//   share 264: 32 heads x  4096 keys, 128 clusters, keep 1/4   19.1 / 15.5
//   share 320: 32 heads x  4990 keys, 200 clusters, keep 1/8   18.0 / 15.3
//   share 520: 32 heads x  8192 keys, 256 clusters, keep 1/8   19.5 / 20.5
//   share 589: 56 heads x  5000 keys, 250 clusters, keep 1/8   19.7 / 20.9
int decode_small_splits(int rows, int L, int C, int U)
{
    if (C > DS_MAX_C || rows > DS_MAX_ROWS) return 0;
    const int splits = std::clamp(DS_GRID / rows, 1, DS_MAX_SPLITS);
    return ((long long)L + U + splits - 1) / splits <= DS_MAX_SHARE ? splits : 0;
}

hipError_t launch_decode_small(const void *q, const void *centroids, const int32_t *sizes, const int32_t *offsets,
                               const float *thresh, const void *Kf, const void *Vf, const void *Ku, const void *Vu,
                               uint32_t *keep_mask, int32_t *n_keys, float *partials, void *out, float *lse, int rows,
                               int H, int G, int L, int C, int U, int splits, float sm_scale, hipStream_t s)
{
    if (splits < 1 || splits != decode_small_splits(rows, L, C, U)) return hipErrorInvalidValue;
    hipEvent_t ev0, ev1;
    const dim3 grid(rows * splits);
#define SQ_SMALL_ARGS                                                                                                  \
    (const _Float16 *)q, (const _Float16 *)centroids, sizes, offsets, thresh, (const _Float16 *)Kf, (const _Float16 *)Vf, \
        (const _Float16 *)Ku, (const _Float16 *)Vu, keep_mask, n_keys, partials, rows, H, G, L, C, U, splits, sm_scale
    if (profile_pair(&ev0, &ev1))
        hipExtLaunchKernelGGL(decode_small_kernel, grid, dim3(256), 0, s, ev0, ev1, 0, SQ_SMALL_ARGS);
    else
        hipLaunchKernelGGL(decode_small_kernel, grid, dim3(256), 0, s, SQ_SMALL_ARGS);
#undef SQ_SMALL_ARGS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(decode_small_merge_kernel, dim3(rows), dim3(MERGE_THREADS), 0, s, partials, (_Float16 *)out, lse,
                       splits);
    return hipGetLastError();
}

}  // namespace sq
