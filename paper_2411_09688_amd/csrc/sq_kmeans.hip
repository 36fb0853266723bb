// Offline clustering of the fixed-context keys (Section 3.1): K-means on NORMALISED key vectors, the centroid of
// a cluster being the mean of its vectors.  One call makes one Lloyd iteration:
//
//   half norms  hn_c = |c|^2 / 2 of the current centres                         (one wave per centre)
//   assignment  a(x) = argmin_c |x - c|^2 = argmax_c (x . c - hn_c)              (matrix cores, below)
//   grouping    stable counting sort of the key indices by centre id: per-part histograms (left by the assignment's workgroups
//               up to 32768 keys and 2^23 counts), a scan over parts and centres, and a scatter in key order -- sizes, offsets and the member
//               list of every cluster
//   update      centre = mean of its members' vectors (a cluster without members keeps its centre)
//
// and a last call turns an assignment into what the online path reads: keys and values reordered so that each
// cluster is contiguous, and the centroid of every cluster as the mean of its RAW keys.
//
// The assignment is the only dense contraction: S^T = C X^T on 16x16x32 fp16 MFMA tiles, A = 16 centres read
// from LDS, B = 16 key vectors held in registers.  A wave holds four B sets (64 keys), so every A operand read
// feeds four MFMAs; the four waves of a workgroup (256 keys) share the centre stream, which travels from global memory
// straight into one of three LDS stages, two groups of 64 centres ahead, one barrier per group.  A lane
// owns one key per B set and four consecutive centres per tile; it keeps the best four it has seen, and which of them it was is
// settled at the end.  The four lane groups are combined last.  Ties go to the lowest centre index: a lane
// visits its centres in ascending order and replaces only on a strictly larger score, and the final combination
// prefers the lower index on equal scores.
// Bound by issue: a workgroup's 16 groups of 1024 matrix cycles each take 36 us at 1.84 GHz, three waves per SIMD 4150 cycles of
// which 3072 are products (74 %; over the whole launch the counters have the matrix cores busy for 68 %, with 2.3 vector
// instructions per score beside the products: 1.9 in the loop, the rest addresses of the loads and the start); 16x16x32 products draw less power than 32x32x16 (1.95 against 1.68 PFLOP/s in a loop of nothing
// else).  32 heads x 32768 keys x 1024 centres: 281 -> 242 us traced on the same card, where compares and selects were three per
// centre and key instead of 1.75 (seven for four), went through padded rows written from registers, and waited for every group at its barrier; with
// products and compares left in the compiler's order 252.
#include <algorithm>
#include <cstddef>

#include "sq_common.hpp"
#include "sq_internal.hpp"

namespace sq {

constexpr int KM_G = 64;                     // centres per staged group
constexpr int KM_RW = 4;                     // B sets (16 keys each) per wave
constexpr int KM_ROWS_PER_WG = 4 * 16 * KM_RW;
constexpr int KM_FUSED_PARTS = 128;          // parts (of a workgroup's keys) whose histograms the assignment leaves, at most
constexpr int KM_STAGES = 3;                 // groups in LDS: one read, two on their way

// Rows of 256 B without padding, filled by the load-to-LDS instruction; the 16-byte chunk c of row r lies at slot c ^ (r % 16), so
// that 16 rows read at one chunk index fall into all banks.
struct KmStage {
    _Float16 Ct[KM_G * D];
    float nhn[KM_G];                         // minus the half norms: the accumulators' starting values
};

// x / |x| per row (fp32 arithmetic), one wave per row; a zero row stays zero.
__global__ __launch_bounds__(256) void normalize_rows_kernel(const _Float16 *__restrict__ K, _Float16 *__restrict__ X,
                                                             size_t rows)
{
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const h2 v = reinterpret_cast<const h2 *>(K + row * D)[lane];
    const float a = (float)v[0], b = (float)v[1];
    const float ss = wave_sum(a * a + b * b);
    const float inv = ss > 0.0f ? 1.0f / sqrtf(ss) : 0.0f;
    h2 o;
    o[0] = (_Float16)(a * inv);
    o[1] = (_Float16)(b * inv);
    reinterpret_cast<h2 *>(X + row * D)[lane] = o;
}

// Minus half the squared norm of every row: 16 lanes per row.  (The sum runs in wave_sum's order, a lane standing for four.)
__global__ __launch_bounds__(256) void half_norm_kernel(const _Float16 *__restrict__ cent, float *__restrict__ nhn,
                                                        int rows)
{
    const int row = blockIdx.x * 16 + (threadIdx.x >> 4), l16 = threadIdx.x & 15;
    const h8 v = reinterpret_cast<const h8 *>(cent + (size_t)min(row, rows - 1) * D)[l16];
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = (float)v[2 * j], b = (float)v[2 * j + 1];
        t[j] = a * a + b * b;
    }
    float ss = (t[0] + t[1]) + (t[2] + t[3]);
    ss += dpp_f<0xb1>(ss);
    ss += dpp_f<0x4e>(ss);
    ss += dpp_f<0x141>(ss);
    ss += dpp_f<0x140>(ss);
    if (l16 == 0 && row < rows) nhn[row] = -(0.5f * ss);
}

// HIST: the workgroup's keys are a part of the grouping below, and it leaves their histogram, too: 16 bits a centre in a row of Cs.
template <bool HIST>
__global__ __launch_bounds__(256, 3) void kmeans_assign_kernel(const _Float16 *__restrict__ X,
                                                               const _Float16 *__restrict__ cent,
                                                               const float *__restrict__ nhn,
                                                               int32_t *__restrict__ assign, uint32_t *__restrict__ hist,
                                                               int L, int C, int Cs)
{
    __shared__ __align__(16) KmStage stage[KM_STAGES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kg = lane >> 4;
    const int h = blockIdx.y;
    const int r0 = (blockIdx.x * 4 + wave) * 16 * KM_RW;      // first key of this wave (may lie past the end)
    const int ng = (C + KM_G - 1) / KM_G;

    // A group: 16 pieces of four rows, four per wave; the half norms by wave 0.  Centres past the end repeat the last one, whose
    // index is lower, so they are never best.
    const char *ch = reinterpret_cast<const char *>(cent + (size_t)h * C * D);
    const float *hh = nhn + (size_t)h * C;
    typedef __attribute__((address_space(3))) void *lptr_t;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lptr_t)stage);
    auto fetch = [&](int g, int st) {
        const uint32_t lds = lds0 + (uint32_t)(st * sizeof(KmStage));
        if (wave == 0)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds + (uint32_t)offsetof(KmStage, nhn)),
                         "v"((uint32_t)min(g * KM_G + lane, C - 1) * 4u), "s"(hh) : "m0", "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = (wave * 4 + i) * 4 + kg;            // row of the group; r % 16 = 4 i + kg
            const uint32_t at = (uint32_t)min(g * KM_G + r, C - 1) * 256u + (uint32_t)((lane & 15) ^ (4 * i + kg)) * 16u;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds + (uint32_t)((wave * 4 + i) * 1024)),
                         "v"(at), "s"(ch) : "m0", "memory");
        }
    };
    fetch(0, 0);
    if (ng > 1) fetch(1, 1);
    h8 bx[KM_RW][4];
#pragma unroll
    for (int r = 0; r < KM_RW; ++r) {
        const int row = min(r0 + r * 16 + col, L - 1);        // keys past the end repeat the last one
        const h8 *xp = reinterpret_cast<const h8 *>(X + ((size_t)h * L + row) * D);
#pragma unroll
        for (int s = 0; s < 4; ++s) bx[r][s] = xp[s * 4 + kg];
    }

    // The running best of a lane's centres, four consecutive ones (a tile's rows kg * 4 ..) at a time: the largest score, the first
    // of the four that reached it first, and their scores but the last one's, which tell at the end which of the four it was.
    // Seven instructions per four centres and key, where a compare and two selects per centre were twelve.
    float best[KM_RW], sv[KM_RW][3];
    int bi[KM_RW];
#pragma unroll
    for (int r = 0; r < KM_RW; ++r) {
        best[r] = SQ_NEG_INF;
        bi[r] = 0;
#pragma unroll
        for (int v = 0; v < 3; ++v) sv[r][v] = SQ_NEG_INF;
    }
    uint32_t rd[4];                                           // operand of step s: row col of a tile, chunk 4 s + kg
#pragma unroll
    for (int s = 0; s < 4; ++s) rd[s] = (uint32_t)(col * 256 + ((s * 4 + kg) ^ col) * 16);
    // Scores of tile u of a staged group: acc[r][v] = x_r . c - hn_c for c = u*16 + kg*4 + v (the accumulator starts
    // at -hn_c).
    auto tile = [&](const KmStage &st, int u, f4 (&acc)[KM_RW]) {
        const f4 nh = *reinterpret_cast<const f4 *>(st.nhn + u * 16 + kg * 4);
        const char *rows = reinterpret_cast<const char *>(st.Ct) + u * 4096;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const h8 a = *reinterpret_cast<const h8 *>(rows + rd[s]);
#pragma unroll
            for (int r = 0; r < KM_RW; ++r)
                acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bx[r][s], s == 0 ? nh : acc[r], 0, 0, 0);
        }
    };
    auto take = [&](const f4 (&acc)[KM_RW], int c0) {
        float m[KM_RW];
        bool win[KM_RW];
#pragma unroll
        for (int r = 0; r < KM_RW; ++r) m[r] = fmaxf(fmaxf(fmaxf(fmaxf(best[r], acc[r][0]), acc[r][1]), acc[r][2]), acc[r][3]);
#pragma unroll
        for (int r = 0; r < KM_RW; ++r) win[r] = m[r] > best[r];
#pragma unroll
        for (int r = 0; r < KM_RW; ++r) {
            bi[r] = win[r] ? c0 : bi[r];
#pragma unroll
            for (int v = 0; v < 3; ++v) sv[r][v] = win[r] ? acc[r][v] : sv[r][v];
            best[r] = m[r];
        }
    };
    // The running best is updated one tile behind the matrix cores: the compares of a tile come after the MFMAs of
    // the next one in program order, which lets the compiler interleave the two kinds of work.
    f4 cur[KM_RW];
#pragma unroll
    for (int r = 0; r < KM_RW; ++r) cur[r] = f4{SQ_NEG_INF, SQ_NEG_INF, SQ_NEG_INF, SQ_NEG_INF};
    int cur_c0 = 0, st = 0;
    for (int g = 0; g < ng; ++g) {
        // Group g has landed when the loads of group g + 1 alone (four rows' pieces; none behind the last group) are under way;
        // behind the barrier that holds for all waves, and group g - 1 has been read by all of them.
        if (g + 1 < ng) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (g + 2 < ng) fetch(g + 2, st == 0 ? 2 : st - 1);
        const KmStage &cs = stage[st];
#pragma unroll
        for (int u = 0; u < KM_G / 16; ++u) {
            f4 nxt[KM_RW];
            tile(cs, u, nxt);
            take(cur, cur_c0);
#pragma unroll
            for (int r = 0; r < KM_RW; ++r) cur[r] = nxt[r];
            cur_c0 = g * KM_G + u * 16 + kg * 4;
#pragma unroll
            for (int i = 0; i < 16; ++i) {                    // (products and compares alternate)
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            }
        }
        st = st == 2 ? 0 : st + 1;
    }
    take(cur, cur_c0);
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(stage);    // two centres a word, where the groups were
    const int words = Cs >> 1;
    if constexpr (HIST) {
        static_assert(sizeof(stage) >= SELECT_MAX_C * 2, "a count of 16 bits for every centre");
        __syncthreads();                                      // (the last group is read)
        for (int w = tid; w < words; w += 256) s_cnt[w] = 0u;
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < KM_RW; ++r) {
        bi[r] += sv[r][0] == best[r] ? 0 : sv[r][1] == best[r] ? 1 : sv[r][2] == best[r] ? 2 : 3;
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float so = __shfl_xor(best[r], off);
            const int io = __shfl_xor(bi[r], off);
            if (so > best[r] || (so == best[r] && io < bi[r])) {
                best[r] = so;
                bi[r] = io;
            }
        }
        const int row = r0 + r * 16 + col;
        if (kg == 0 && row < L) {
            assign[(size_t)h * L + row] = bi[r];
            const int c = min(bi[r], C - 1);                  // (clamped like an id that is read back)
            if (HIST) atomicAdd(&s_cnt[c >> 1], 1u << (16 * (c & 1)));   // (at most 256 a centre)
        }
    }
    if constexpr (HIST) {
        __syncthreads();
        uint32_t *dst = hist + ((size_t)h * gridDim.x + blockIdx.x) * words;
        for (int w = tid; w < words; w += 256) dst[w] = s_cnt[w];
    }
}

// Grouping, step 1: histogram of centre ids over one part of a head's keys.  (Where the assignment did not leave it.)
__global__ __launch_bounds__(256) void kmeans_hist_kernel(const int32_t *__restrict__ assign, int32_t *__restrict__ hist,
                                                          int L, int C, int PL, int P)
{
    extern __shared__ int s_cnt[];
    const int p = blockIdx.x, h = blockIdx.y;
    for (int c = threadIdx.x; c < C; c += 256) s_cnt[c] = 0;
    __syncthreads();
    const int k_end = min(L, (p + 1) * PL);
    for (int k = p * PL + threadIdx.x; k < k_end; k += 256)      // (an id out of range counts for the nearest valid one)
        atomicAdd(&s_cnt[min(max(assign[(size_t)h * L + k], 0), C - 1)], 1);
    __syncthreads();
    int32_t *dst = hist + ((size_t)h * P + p) * C;
    for (int c = threadIdx.x; c < C; c += 256) dst[c] = s_cnt[c];
}

// Grouping, step 2: per centre, the part counts become exclusive prefixes over the parts and their total the cluster size.  A
// workgroup takes 64 centres, each of its four waves a quarter of the parts (at most 64, see kmeans_part_len, or 128 of 16 bits).  5.8 us at 32 heads x
// 1024 centres x 64 parts, where one workgroup per head, which also scanned the sizes into offsets, took 9.4.
// CT: type of the counts, 16 bits where the keys of a head are at most 2^15 in at most 128 parts.  Cs: counts of a part's row.
template <typename CT>
__global__ __launch_bounds__(256) void kmeans_scan_kernel(CT *__restrict__ hist, int32_t *__restrict__ sizes, int C, int Cs, int P)
{
    constexpr int KM_SCAN_PARTS = sizeof(CT) == 2 ? KM_FUSED_PARTS / 4 : 16;
    __shared__ int s_tot[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane, h = blockIdx.y;
    const int per = (P + 3) >> 2, p0 = wave * per, n = max(0, min(per, P - p0));
    CT *col = hist + ((size_t)h * P + p0) * Cs + min(c, C - 1);
    int t[KM_SCAN_PARTS], sum = 0;
#pragma unroll
    for (int u = 0; u < KM_SCAN_PARTS; ++u) t[u] = u < n ? (int)col[(size_t)u * Cs] : 0;
#pragma unroll
    for (int u = 0; u < KM_SCAN_PARTS; ++u) sum += t[u];
    s_tot[wave][lane] = sum;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int v = s_tot[w][lane];
        if (w < wave) before += v;
        total += v;
    }
    if (c >= C) return;
#pragma unroll
    for (int u = 0; u < KM_SCAN_PARTS; ++u) {
        if (u < n) col[(size_t)u * Cs] = (CT)before;
        before += t[u];
    }
    if (wave == 0) sizes[(size_t)h * C + c] = total;
}

// Grouping, step 3: one WAVE per part walks the part's keys in index order, 64 at a time.  The lanes that hold the
// same centre id are found in registers (a ballot per bit of the id); a lane's slot is the cluster's cursor plus the number of matching lanes below it, so members appear in
// ascending key order inside every cluster (a stable sort).  The cursors live in LDS and are touched by this one
// wave only, in program order (all lanes of a group read the cursor, then its last lane advances it): no atomics.
// The launch is one wave's chain of reads, so the ids of 512 keys are fetched together, the first ones before the sizes are
// scanned, and the sizes of 1024 centres.  The parts of a head share an XCD: they fill the same lines of the list, which would
// otherwise lie in eight L2s, a few words in each.  Whole iteration of 32 heads x 32K keys x 1024 centres 299.4 -> 294.2 us (scatter
// 17.0 -> 12.0 traced; with the XCDs alone 295.8, with the reads alone 298.9), 16 heads x 30000 x 800 139.4 -> 137.1, one head x 20000
// x 500 35.0 -> 34.6.
constexpr int KM_SCATTER_AHEAD = 8, KM_CURSOR_AHEAD = 16;
template <typename CT>
__global__ __launch_bounds__(64) void kmeans_scatter_kernel(const int32_t *__restrict__ assign,
                                                            const CT *__restrict__ hist,
                                                            const int32_t *__restrict__ sizes, int32_t *__restrict__ offsets,
                                                            int32_t *__restrict__ perm, int H, int L, int C, int Cs, int PL, int P)
{
    extern __shared__ int s_cur[];
    const int per_xcd = (H * P + 7) >> 3, unit = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (unit >= H * P) return;
    const int h = unit / P, p = unit - h * P, lane = threadIdx.x;
    const CT *hp = hist + ((size_t)h * P + p) * Cs;
    const int32_t *np = sizes + (size_t)h * C;
    int32_t *op = offsets + (size_t)h * (C + 1);
    // Where the part's members of every centre go: the sizes of the centres in front -- scanned by every wave, 64 centres at a
    // time with sixteen such loads under way; the first part's wave writes them as the offsets -- and the members in parts in front.
    const int k_end = min(L, (p + 1) * PL);
    const int32_t *ap = assign + (size_t)h * L;
    int ids[KM_SCATTER_AHEAD];                             // of a stretch of keys, all of them under way before the first is used
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < KM_SCATTER_AHEAD; ++u) ids[u] = ap[min(k0 + u * 64 + lane, L - 1)];
    };
    fetch(p * PL);
    int carry = 0;
    for (int c0 = 0; c0 < C; c0 += 64 * KM_CURSOR_AHEAD) {
        int n[KM_CURSOR_AHEAD], before[KM_CURSOR_AHEAD];
#pragma unroll
        for (int u = 0; u < KM_CURSOR_AHEAD; ++u) {
            const int c = min(c0 + u * 64 + lane, C - 1);
            n[u] = np[c];
            before[u] = (int)hp[c];
        }
#pragma unroll
        for (int u = 0; u < KM_CURSOR_AHEAD; ++u) {
            if (c0 + u * 64 >= C) break;                   // uniform
            n[u] = c0 + u * 64 + lane < C ? n[u] : 0;
            const int c = c0 + u * 64 + lane, incl = wave_inclusive_scan(n[u], lane), off = carry + incl - n[u];
            if (c < C) {
                s_cur[c] = off + before[u];
                if (p == 0) op[c] = off;
            }
            carry += __builtin_amdgcn_readlane(incl, 63);
        }
    }
    if (p == 0 && lane == 0) op[C] = L;
    __syncthreads();
    const int nbits = 32 - __clz(max(C - 1, 1));           // bits of a centre id
    for (int k0 = p * PL; k0 < k_end; k0 += 64 * KM_SCATTER_AHEAD) {
        if (k0 > p * PL) fetch(k0);
#pragma unroll
        for (int u = 0; u < KM_SCATTER_AHEAD; ++u) {
            if (k0 + u * 64 >= k_end) break;               // uniform
            const int k = k0 + u * 64 + lane;
            const bool valid = k < k_end;
            const int c = valid ? min(max(ids[u], 0), C - 1) : -1;   // clamped like the counts
            // Lanes with the same centre id, found bit by bit: a lane keeps the lanes that agree with it on every bit of
            // the id (one ballot per bit, no data-dependent loop).
            uint64_t m = __ballot(valid);
            for (int b = 0; b < nbits; ++b) {              // uniform trip count
                const bool bit = (c >> b) & 1;
                const uint64_t bal = __ballot(valid && bit);
                m &= bit ? bal : ~bal;
            }
            const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const int cnt = __popcll(m);
            if (valid) {
                const int cur = s_cur[c];
                if (rank == cnt - 1) s_cur[c] = cur + cnt;
                perm[(size_t)h * L + cur + rank] = k;
            }
        }
    }
}

// Mean of the rows of `src` listed for each cluster (members perm[off .. off + n) of head h), fp32 accumulation in
// a fixed order: 16 member slots x 16 sixteen-byte pieces of a row, then the slots are added in ascending order.
// An empty cluster copies prev (the centre it had) or, with prev == NULL, writes zeros.  perm == NULL: the members of
// a cluster are the rows off .. off + n themselves.
// A gather bound by how many rows are under way: offset, index and row are three dependent reads.  So a workgroup takes
// CM_CLUSTERS consecutive clusters, whose indices (one stretch of perm) it fetches together, and requests the first 32 rows of the
// next cluster before it folds the current one's.  The heads are taken last to first: what the assignment read last is still in the
// last-level cache.  32 heads x 32768 keys x 1024 centres, traced: one cluster per workgroup 72 us before, 66 in this form, four 55,
// eight 60; eight with the heads first to last 68.  Few clusters in all are spread over more workgroups (4096, if there are as many).
constexpr int CM_CLUSTERS = 4, CM_CAP = 512;                 // at most; indices in LDS, the rest of a longer stretch is read from memory
__global__ __launch_bounds__(256) void cluster_mean_kernel(const _Float16 *__restrict__ src,
                                                           const int32_t *perm,
                                                           const int32_t *__restrict__ sizes,
                                                           const int32_t *__restrict__ offsets,
                                                           const _Float16 *prev, _Float16 *out, int L, int C, int per)
{
    __shared__ float s_acc[2][16][D + 4];
    __shared__ int s_mem[CM_CAP], s_off[CM_CLUSTERS], s_n[CM_CLUSTERS];
    const int h = (int)(gridDim.y - 1 - blockIdx.y), c0 = (int)blockIdx.x * per, tid = threadIdx.x;
    const int slot = tid >> 4, piece = tid & 15, nc = min(per, C - c0);
    if (tid < CM_CLUSTERS) {
        const int c = min(c0 + tid, C - 1), off = min(max(offsets[(size_t)h * (C + 1) + c], 0), L);
        s_off[tid] = off;
        s_n[tid] = min(max(sizes[(size_t)h * C + c], 0), L - off);
    }
    __syncthreads();
    const int32_t *mem = perm ? perm + (size_t)h * L : nullptr;
    const int m0 = s_off[0];
    int held = 0;                                             // indices in LDS (one cluster: they are read where they are used)
    if (mem && per > 1) {
        held = __builtin_amdgcn_readfirstlane(min(s_off[nc - 1] + s_n[nc - 1] - m0, CM_CAP));
        for (int i = tid; i < held; i += 256) s_mem[i] = mem[m0 + i];
        __syncthreads();
    }
    const _Float16 *rows = src + (size_t)h * L * D;
    auto row_of = [&](int pos) {                              // member at position pos of the head's list
        int r = pos;
        if (mem) {
            const int i = pos - m0;
            r = i >= 0 && i < held ? s_mem[i] : mem[pos];     // (clusters in another order may lie outside the stretch)
        }
        return *reinterpret_cast<const h8 *>(rows + (size_t)min(max(r, 0), L - 1) * D + piece * 8);
    };
    const h8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    h8 a = zero, b = zero;                                    // the current cluster's rows of this slot: slot, slot + 16
    auto first_rows = [&](int i) {
        const int off = s_off[i], n = s_n[i];
        a = slot < n ? row_of(off + slot) : zero;
        b = slot + 16 < n ? row_of(off + slot + 16) : zero;
    };
    first_rows(0);
    for (int i = 0; i < nc; ++i) {                            // (workgroup-uniform)
        const int off = s_off[i], n = s_n[i];
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.0f + (float)a[j];
        if (slot + 16 < n)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (float)b[j];
        if (i + 1 < nc) first_rows(i + 1);
        int m = slot + 32;
        for (; m + 16 < n; m += 32) {                         // two rows in flight
            const h8 v = row_of(off + m), w = row_of(off + m + 16);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (float)v[j];
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (float)w[j];
        }
        if (m < n) {
            const h8 v = row_of(off + m);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += (float)v[j];
        }
        float (&buf)[16][D + 4] = s_acc[i & 1];
#pragma unroll
        for (int j = 0; j < 8; ++j) buf[slot][piece * 8 + j] = acc[j];
        __syncthreads();                                      // (the other buffer is read before the next one)
        if (tid < D) {
            const size_t at = ((size_t)h * C + c0 + i) * D + tid;
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k < 16; ++k) s += buf[k][tid];
            out[at] = n > 0 ? (_Float16)(s / (float)n) : prev ? prev[at] : (_Float16)0.0f;
        }
    }
}

static hipError_t launch_cluster_mean(const void *src, const int32_t *perm, const int32_t *sizes, const int32_t *offsets,
                                      const void *prev, void *out, int H, int L, int C, hipStream_t s)
{
    const int per = (int)std::clamp((long long)H * C / 4096, 1ll, (long long)CM_CLUSTERS);
    hipLaunchKernelGGL(cluster_mean_kernel, dim3((C + per - 1) / per, H), dim3(256), 0, s, (const _Float16 *)src, perm, sizes,
                       offsets, (const _Float16 *)prev, (_Float16 *)out, L, C, per);
    return hipGetLastError();
}

// dst[h, i, :] = src[h, perm[h, i], :] for up to two tensors (blockIdx.z), 16 rows per workgroup.
__global__ __launch_bounds__(256) void gather_rows_kernel(const _Float16 *__restrict__ src0, _Float16 *__restrict__ dst0,
                                                          const _Float16 *__restrict__ src1, _Float16 *__restrict__ dst1,
                                                          const int32_t *__restrict__ perm, int L)
{
    const int h = blockIdx.y;
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), piece = threadIdx.x & 15;
    if (i >= L) return;
    const _Float16 *src = blockIdx.z ? src1 : src0;
    _Float16 *dst = blockIdx.z ? dst1 : dst0;
    const int k = min(max(perm[(size_t)h * L + i], 0), L - 1);
    *reinterpret_cast<h8 *>(dst + ((size_t)h * L + i) * D + piece * 8) =
        *reinterpret_cast<const h8 *>(src + ((size_t)h * L + k) * D + piece * 8);
}

static int kmeans_part_len(int L)
{
    const int want = (L + 63) / 64;                           // at most 64 parts per head
    const int pl = ((want + 255) / 256) * 256;
    return pl < 512 ? 512 : pl;
}

// Counts of a part's row of 16 bits: whole lines of 128 bytes, since workgroups on different XCDs write neighbouring rows (rows of C,
// whole steps, us, rows of C / of lines: 32 heads x 32768 keys x 1638 centres 429.0 / 419.2, x 1900 484.0 / 472.9, 8 x 32768 x 6553
// 414.4 / 407.6, 24 x 32768 x 1638 328.7 / 322.6; with the launch that counted the ids again 428.3, 479.2, 417.7, 327.9).
// Below 256 centres the rows are a small part of the step and the lines would be mostly padding.
static int kmeans_hist_row(int C) { return C < 256 ? (C + 1) & ~1 : (C + 63) & ~63; }

// Does the assignment leave the histograms?  The launch that counted the ids again is a launch's time where there is little to count;
// what it costs the assignment is a microsecond a workgroup, under the others' products, and the rows of 256 keys in 16 bits are as many
// bytes as those of 512 in 32.  Whole step, us, with that launch / here: 32 heads x 32768 keys x 1024 centres 287.1 / 283.2, 16 x 30000 x
// 800 129.9 / 127.0, 4 x 32768 x 1638 79.0 / 75.7, 1 x 20000 x 500 34.0 / 30.4, 32 x 3000 x 130 35.4 / 32.1, 1 x 2000 x 40 23.1 / 20.0.
// The lines are the scan's 128 parts (and every prefix has to fit 16 bits), and 2^23 counts (16 MB): with more they leave the L2s before
// they are read, 8 x 32768 x 8192 506.5 / 499.1, 4 x 32768 x 16384 522 / 515, 32 x 32768 x 2048 505.5 / 501.7, but
// 32 x 32768 x 4096 933 / 943, 16 x 32768 x 6000 706 / 722, 12 x 32768 x 8192 719 / 728, 6 x 32768 x 16384 738 / 764.
static bool kmeans_fused(int heads, int L, int C)
{
    const long long parts = (L + KM_ROWS_PER_WG - 1) / KM_ROWS_PER_WG;
    return parts <= KM_FUSED_PARTS && heads * parts * kmeans_hist_row(C) <= 1ll << 23;
}

size_t kmeans_hist_ints(int heads, int L, int C)
{
    const size_t PL = kmeans_part_len(L), counted = (size_t)heads * ((L + PL - 1) / PL) * C;   // (cluster_nest counts them always)
    if (!kmeans_fused(heads, L, C)) return counted;
    return std::max(counted, (size_t)heads * ((L + KM_ROWS_PER_WG - 1) / KM_ROWS_PER_WG) * kmeans_hist_row(C) / 2);
}

hipError_t launch_normalize_rows(const void *K, void *X, size_t rows, hipStream_t s)
{
    hipLaunchKernelGGL(normalize_rows_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, (const _Float16 *)K,
                       (_Float16 *)X, rows);
    return hipGetLastError();
}

// Stable grouping of the rows by centre id: sizes, offsets and the member list of every centre.
template <typename CT>
static void launch_scan_scatter(const int32_t *assign, int32_t *sizes, int32_t *offsets, int32_t *perm, CT *hist, int H, int L, int C,
                                int Cs, int PL, hipStream_t s)
{
    const int P = (L + PL - 1) / PL;
    hipLaunchKernelGGL(kmeans_scan_kernel<CT>, dim3((C + 63) / 64, H), dim3(256), 0, s, hist, sizes, C, Cs, P);
    hipLaunchKernelGGL(kmeans_scatter_kernel<CT>, dim3((H * P + 7) / 8 * 8), dim3(64), (size_t)C * 4, s, assign, (const CT *)hist,
                       (const int32_t *)sizes, offsets, perm, H, L, C, Cs, PL, P);
}

static void launch_group(const int32_t *assign, int32_t *sizes, int32_t *offsets, int32_t *perm, int32_t *hist, int H,
                         int L, int C, hipStream_t s)
{
    const int PL = kmeans_part_len(L), P = (L + PL - 1) / PL;
    hipLaunchKernelGGL(kmeans_hist_kernel, dim3(P, H), dim3(256), (size_t)C * 4, s, assign, hist, L, C, PL, P);
    launch_scan_scatter(assign, sizes, offsets, perm, hist, H, L, C, C, PL, s);
}

hipError_t launch_kmeans_step(const void *X, const void *centers_in, void *centers_out, int32_t *assign,
                              int32_t *sizes, int32_t *offsets, int32_t *perm, float *hn, int32_t *hist, int H, int L,
                              int C, hipStream_t s)
{
    hipLaunchKernelGGL(half_norm_kernel, dim3((H * C + 15) / 16), dim3(256), 0, s, (const _Float16 *)centers_in, hn, H * C);
    const dim3 grid_a((L + KM_ROWS_PER_WG - 1) / KM_ROWS_PER_WG, H);
    const bool fused = kmeans_fused(H, L, C);
    auto assign_kernel = [&](auto kernel) {
        hipEvent_t ev0, ev1;
        if (profile_pair(&ev0, &ev1))
            hipExtLaunchKernelGGL(kernel, grid_a, dim3(256), 0, s, ev0, ev1, 0, (const _Float16 *)X, (const _Float16 *)centers_in,
                                  (const float *)hn, assign, reinterpret_cast<uint32_t *>(hist), L, C, kmeans_hist_row(C));
        else
            hipLaunchKernelGGL(kernel, grid_a, dim3(256), 0, s, (const _Float16 *)X, (const _Float16 *)centers_in, (const float *)hn,
                               assign, reinterpret_cast<uint32_t *>(hist), L, C, kmeans_hist_row(C));
    };
    if (fused) {
        assign_kernel(kmeans_assign_kernel<true>);
        launch_scan_scatter(assign, sizes, offsets, perm, reinterpret_cast<uint16_t *>(hist), H, L, C, kmeans_hist_row(C), KM_ROWS_PER_WG, s);
    } else {
        assign_kernel(kmeans_assign_kernel<false>);
        launch_group(assign, sizes, offsets, perm, hist, H, L, C, s);
    }
    return launch_cluster_mean(X, perm, sizes, offsets, centers_in, centers_out, H, L, C, s);
}

// Nesting fine clusters under coarse ones (Section 3.3: the coarse level is a clustering of the fine centroids).
// perm_coarse lists the fine cluster ids grouped by coarse cluster; the fine clusters are renumbered in that order
// (inv[old id] = new id), every key's cluster id is translated, and the keys are grouped again.
__global__ __launch_bounds__(256) void invert_perm_kernel(const int32_t *__restrict__ perm, int32_t *__restrict__ inv,
                                                          int n)
{
    const int h = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const int f = perm[(size_t)h * n + j];
    if ((unsigned)f < (unsigned)n) inv[(size_t)h * n + f] = j;     // (a value out of range is ignored)
}

__global__ __launch_bounds__(256) void relabel_kernel(const int32_t *__restrict__ assign, const int32_t *__restrict__ inv,
                                                      int32_t *__restrict__ assign_new, int L, int C)
{
    const int h = blockIdx.y, k = blockIdx.x * 256 + threadIdx.x;
    if (k >= L) return;
    const int a = min(max(assign[(size_t)h * L + k], 0), C - 1);        // ids are clamped into range, so that malformed
    assign_new[(size_t)h * L + k] = min(max(inv[(size_t)h * C + a], 0), C - 1);   // input cannot index out of bounds later
}

// Keys under each coarse cluster: its children are fine clusters child_offsets[j] .. child_offsets[j+1]-1.
__global__ __launch_bounds__(256) void coarse_sizes_kernel(const int32_t *__restrict__ offsets_fine,
                                                           const int32_t *__restrict__ child_offsets,
                                                           int32_t *__restrict__ sizes_coarse, int C1, int C2)
{
    const int h = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= C1) return;
    const int32_t *co = child_offsets + (size_t)h * (C1 + 1), *of = offsets_fine + (size_t)h * (C2 + 1);
    const int lo = min(max(co[j], 0), C2), hi = min(max(co[j + 1], lo), C2);
    sizes_coarse[(size_t)h * C1 + j] = of[hi] - of[lo];
}

hipError_t launch_cluster_nest(const int32_t *assign_fine, const int32_t *perm_coarse, const int32_t *child_offsets,
                               int32_t *assign_new, int32_t *sizes, int32_t *offsets, int32_t *perm,
                               int32_t *sizes_coarse, int32_t *inv, int32_t *hist, int H, int L, int C2, int C1,
                               hipStream_t s)
{
    hipLaunchKernelGGL(invert_perm_kernel, dim3((C2 + 255) / 256, H), dim3(256), 0, s, perm_coarse, inv, C2);
    hipLaunchKernelGGL(relabel_kernel, dim3((L + 255) / 256, H), dim3(256), 0, s, assign_fine, (const int32_t *)inv,
                       assign_new, L, C2);
    launch_group(assign_new, sizes, offsets, perm, hist, H, L, C2, s);
    hipLaunchKernelGGL(coarse_sizes_kernel, dim3((C1 + 255) / 256, H), dim3(256), 0, s, (const int32_t *)offsets,
                       child_offsets, sizes_coarse, C1, C2);
    return hipGetLastError();
}

hipError_t launch_cluster_layout(const void *K, const void *V, const int32_t *perm, const int32_t *sizes,
                                 const int32_t *offsets, void *K_sorted, void *V_sorted, void *centroids, int H, int L,
                                 int C, hipStream_t s)
{
    if (K_sorted)                                             // (V_sorted == NULL: keys only)
        hipLaunchKernelGGL(gather_rows_kernel, dim3((L + 15) / 16, H, V_sorted ? 2 : 1), dim3(256), 0, s,
                           (const _Float16 *)K, (_Float16 *)K_sorted, (const _Float16 *)V, (_Float16 *)V_sorted, perm, L);
    return launch_cluster_mean(K, perm, sizes, offsets, nullptr, centroids, H, L, C, s);
}

}  // namespace sq
