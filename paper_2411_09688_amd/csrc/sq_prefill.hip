// Prefill-time sparse attention (Section 4.2) with per-query selection: every query token attends to the
// keys of the clusters set in its own keep mask, plus the (causal) user keys, one softmax over the union.
//
// Layout of the computation (FlashAttention-2 style: grid over heads x query blocks x shares of the key blocks, loop over
// key blocks, online softmax), written for CDNA4 matrix cores:
//   * a wave owns 32 queries; a workgroup of eight (or four) waves walks the same 64-key blocks, whose K and V tiles are
//     staged row-major in LDS once per workgroup, straight from global memory with the load-to-LDS instruction;
//   * scores are computed TRANSPOSED, S^T = K Q^T, with 32x32x16 fp16 MFMA tiles (A = 32 keys, B = 32 queries).  In the
//     accumulator layout a lane then owns ONE query column for the whole kernel (and 16 keys per tile; lanes l and l + 32
//     share a column), so the reference maximum, the running sum and the rescaling of the output are per-lane scalars, and
//     P^T is packed into the B operand of the next product in registers, with no cross-lane traffic;
//   * O^T = V^T P^T uses A = V^T tiles read from the row-major V tile with the transposing LDS read
//     (ds_read_b64_tr_b16), so V needs no transposition on its way into LDS;
//   * the loop is pipelined inside a wave: while the softmax of block i runs on the vector ALU, the products S^T of block
//     i + 1 and O^T of block i are issued between its instructions (the order is laid out by hand, a pair of scores at a
//     time).  Two waves per SIMD that run their phases one after the other overlap little of them on this chip, and a wave
//     issues at most one vector instruction per five cycles, so both the overlap and the instruction count matter;
//   * masks cost no vector arithmetic per score: a lane's visible keys of a block are two words (one AND/OR pair per run of
//     keys of one cluster, prepared by a table launch), and the score products start from 0 (visible) or -inf (hidden),
//     four start values per LDS read from a 16-entry table.
//   * a workgroup whose waves need only part of the blocks it lists (neighbouring queries that keep the same clusters) takes the
//     sparse walk instead, in which a wave does a block from scores to output product in one go (see PF_SPARSE_NUM);
//   * outputs that infinite or NaN values made NaN are taken again at the end (prefill_again).
// What it is bound by at 32 heads x 1024 tokens x 32K keys (560 GFLOP executed, padding included): about 3600 cycles per block and
// pair of waves against 2050 of matrix work.  The traced kernel takes 527 to 706 us, 576 on average (the clock follows the load):
// 0.97 PFLOP/s, 1.06 at best, where the library's large fp16 product reaches 1.18 on the same card.  Whole step: 819 us with the
// form before it (16 queries per wave, masks and maxima on every score, phases one after the other), 660 with 32 queries per wave
// in that order, 580 in this one.  Timing-only builds of it: without loads -9 %, without LDS operand reads -11 %, without
// exponentials -12 %, without products -25 % (sum of nothing dominates).
// The user block is causal when causal_user is set (query t sees user keys 0..t); the fixed context is
// always fully visible.
//
// SHARED variant (selection on averaged scores, Appendix D "Prefill Stage"): all query tokens of a (sequence,
// head) attend to ONE kept set.  The kept ranges are expanded into a list of key rows (the key-index tensor of
// Section 4.2); the kernel walks that list 64 keys at a time, gathering K and V rows by index (the indices travel in
// registers ahead of the rows), with no per-query masks: only the tail of the last block and the causal user keys are
// hidden, so every executed tile is useful work.  The step on averaged scores makes the list of a share here (SELECT): where
// prefill_selects() the launch in front that would make it for all of them is left out.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "sq_block_table.hpp"
#include "sq_common.hpp"
#include "sq_internal.hpp"
#include "sq_mean_row.hpp"

namespace sq {

// K and V tiles in LDS: unpadded rows of 256 B, filled straight from global memory by the load-to-LDS instruction
// (global_load_lds_dwordx4: the 64 lanes of a wave write 64 x 16 contiguous bytes = four whole rows), and swizzled
// instead of padded so that the operand reads stay free of bank conflicts: the 16-byte chunk c of row r sits at slot
// c ^ swz(r).  The swizzle is applied on the global side (lane = slot: it fetches chunk slot ^ swz(r)).
//   K (16-byte reads, 16 rows at one chunk index per group of lanes): swz = r % 16 -- the 16 rows land in 16 slots.
//   V (transposing 8-byte reads, 4 rows x 64 bytes per half wave): swz = 4 * (r % 4) -- the four chunks of a row stay
//   together and the four rows land in four different quarters of the banks.
__device__ __forceinline__ int pf_k_swz(int row) { return row & 15; }
__device__ __forceinline__ int pf_v_swz(int row) { return (row & 3) << 2; }

// The block table of a call that has no lookup launch to make it in (sq_sparse_attn_prefill): see sq_block_table.hpp.
__global__ __launch_bounds__(256) void block_table_kernel(BlockTable bt)
{
    block_table_part(bt, blockIdx.y, blockIdx.x, 4);
}

// Kept ranges of every (sequence, head) row -> list of key rows: record (first key, count, keys before) writes
// key_idx[row, before + j] = first + j, clamped into the tensor.  One wave per record at a time, the records of a row
// dealt over the gridDim.y workgroups of the row.
__global__ __launch_bounds__(256) void expand_ranges_kernel(DecodePlan plan, int32_t *__restrict__ key_idx, int L)
{
    const size_t row = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nrec = min(plan.hdr[row].x, plan.rec_cap);
    int32_t *dst = key_idx + row * (size_t)L;
    for (int r = (int)blockIdx.y * 4 + wave; r < nrec; r += 4 * (int)gridDim.y) {
        const int4 rc = plan.rec[row * plan.rec_cap + r];
        for (int j = lane; j < rc.y && rc.z + j < L; j += 64) dst[rc.z + j] = max(0, min(rc.x + j, L - 1));
    }
}

constexpr int PF_LIST_CAP = 4096;         // fixed blocks per workgroup that are listed; a longer share is walked whole
constexpr int PF_UMASK_WORDS = SELECT_MAX_C / 32;

// s_um[v * W + 0..W) = OR of the keep masks of the 32 queries of wave v, v = 0..waves-1, those below Lq, of query rows row0...  Two
// barriers inside, the second at the end.  A mask word of eight queries per item: eight independent loads, one LDS atomic; the first
// item's loads are under way while the words are cleared.
__device__ __forceinline__ void pf_union_masks(uint32_t *s_um, const uint32_t *__restrict__ keep_mask, size_t row0, int q0,
                                               int waves, int Lq, int W, int tid, int threads)
{
    const int items = 4 * waves * W;
    uint32_t m[8];
    int g = 0, w = 0;
    auto load = [&](int idx) {
        g = idx / W;
        w = idx - g * W;
#pragma unroll
        for (int k = 0; k < 8; ++k) m[k] = keep_mask[(row0 + min(q0 + g * 8 + k, Lq - 1)) * W + w];   // (past the end: the last row again)
    };
    if (tid < items) load(tid);
    for (int i = tid; i < waves * W; i += threads) s_um[i] = 0u;
    __syncthreads();
    for (int idx = tid; idx < items; idx += threads) {
        uint32_t acc = 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) acc |= m[k];
        if (q0 + g * 8 < Lq && acc) atomicOr(&s_um[(g >> 2) * W + w], acc);
        if (idx + threads < items) load(idx + threads);
    }
    __syncthreads();
}

// Does a wave whose queries' masks OR to s_um need the block with table entry bi?  (A block that spans more
// cluster ids than the window is not decided here: needed.)
__device__ __forceinline__ bool pf_block_needed(int bi, const uint32_t *s_um, int W)
{
    if (bi < 0) return true;
    if (((bi >> 21) & 127) == 0) return false;                 // no key of the block lies in a cluster
    const int first = bi & 0xffff, w0 = first >> 5;
    const unsigned long long two = ((unsigned long long)(w0 + 1 < W ? s_um[w0 + 1] : 0u) << 32) | s_um[w0];
    const uint32_t present = (2u << ((bi >> 16) & 31)) - 1u;   // local clusters that occur in the block
    return ((uint32_t)(two >> (first & 31)) & present) != 0u;
}

// The masked form walks its blocks in one of two ways, chosen by every workgroup from the keep masks when it lists its blocks.
// Where most waves need most of the listed blocks, the pipelined walk (see the head of the file).  Where a wave needs fewer than
// 3/4 of them -- selections that follow the position or that neighbouring queries share -- the sparse walk: a wave does a block
// it needs from scores to output product in one go and leaves the others out, and with four tiles the blocks of a barrier's
// pair come from the two halves of the list, so that waves of different positions work side by side.  Attention call, us,
// 32 heads x 1024 tokens x 32K keys (256 queries a workgroup), pipelined walk / sparse walk, share of (wave, block) pairs needed:
//   kept clusters in a band of 1/8 per 64 queries 226 / 209 (1/4), per 32 queries 312 / 276 (1/5), per 128 149 / 146 (1/2);
//   1/8 of the clusters anywhere, shared by 64 queries 402 / 335 (0.4), by 16 queries 540 / 460 (0.55); 0.16 554 / 529 (0.65),
//   0.2 568 / 573 (0.75), 0.25 571 / 611 (0.8); by nobody 542 / 636 (1).
constexpr int PF_SPARSE_NUM = 3, PF_SPARSE_DEN = 4;
constexpr int PF_AHEAD = 4;                                 // operands requested from LDS ahead of their product
constexpr int pf_bm(int waves) { return 32 * waves; }       // queries per workgroup

// Key blocks staged in LDS (K and V tiles each).  Two: a barrier per block (with four waves two workgroups share a compute
// unit's LDS).  Four in the masked form with eight waves: a barrier per pair of blocks, and the loads have a pair's time to
// land (32 heads x 1024 tokens x 32K keys: 593 -> 583 us per step); the shared-set form's shares are a tenth as long and lose
// as much in the longer prologue (171 -> 174 us).
constexpr int pf_bufs(bool shared, int waves) { return waves == 8 && !shared ? 4 : 2; }
constexpr uint32_t PF_TILE = PF_BN * D * 2;                 // bytes of a K or V tile
constexpr int PF_TABS = 4;                // block table rows in LDS: the block's whose start values are made and the next ones

// f(0), f(1), ... f(N - 1) with the index a compile-time constant.
template <int N, typename F, int... I>
__host__ __device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__host__ __device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}
#define PF_INLINE __attribute__((always_inline))          // (a lambda left as a call would put what it captures in memory)

// The outputs of queries (the active lanes; lane = query column + 32 g, as in prefill_attn_kernel) from the keys they see alone, key
// by key, for queries with a NaN in their output.  Bound by vector instructions, about 200 per key and wave: 32 heads x 1024 tokens
// x 32K keys with a NaN in every query's reach take 26 ms instead of 0.58 (two keys' loads at a time: 24, four: 68, for spills).
// A function of its own, not inlined: as part of the kernel its code lengthened the walk of workgroups with idle waves (32 heads x
// 150 tokens x 32K keys 175 -> 184 us).  seen_user: user keys the query sees; dst: the query's output, to be multiplied by scale,
// or, with several shares, its 128 partial sums.  The other arguments: see the kernel (uniform ones arrive in vector registers).
// LOCAL: table holds the rows of the share's fixed blocks alone, one after the other.
template <bool SHARED, bool LOCAL>
__device__ __attribute__((noinline)) void prefill_again(const _Float16 *q_row, const char *Kf, const char *Vf, const char *Ku,
                                                        const char *Vu, const uint32_t *mrow, const void *table,
                                                        const int32_t *binfo, void *dst, int split, int n_split, int n_fixed, int U,
                                                        int seen_user, float c2, float mneg, float scale)
{
    const int lane = threadIdx.x & 63, g = lane >> 5;
    h8 bq[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) bq[s] = reinterpret_cast<const h8 *>(q_row)[s * 2 + g];
    f4 o[16];                                               // dimensions 8 i + 4 g + (0..3)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = f4{0.f, 0.f, 0.f, 0.f};
    n_split = __builtin_amdgcn_readfirstlane(n_split);
    n_fixed = __builtin_amdgcn_readfirstlane(n_fixed);
    const int nblk_fixed = (n_fixed + PF_BN - 1) / PF_BN, nblk = nblk_fixed + (__builtin_amdgcn_readfirstlane(U) + PF_BN - 1) / PF_BN;
    int own = 0;                                            // blocks of the share in front of this one
    for (int i = __builtin_amdgcn_readfirstlane(split); i < nblk; i += n_split, ++own) {   // (fixed blocks, then user blocks: dealt as in the kernel)
        const bool user = i >= nblk_fixed;
        const int blk = user ? i - nblk_fixed : i;
        unsigned long long seen = 0ull;                     // bit j: the query sees key j of the block
        if (SHARED || user) {
            const int n = (user ? seen_user : n_fixed) - blk * PF_BN;
            seen = n >= 64 ? ~0ull : (1ull << max(n, 0)) - 1ull;
        } else {
            const uint32_t *rp = static_cast<const uint32_t *>(table) + (size_t)blk * PF_BN;
            for (int k = 0; k < ((binfo[blk] >> 21) & 127); ++k) {
                const uint32_t c = rp[k] & 0xffffu;
                if ((mrow[c >> 5] >> (c & 31u)) & 1u) seen |= (~0ull >> (63 - (int)((rp[k] >> 22) & 63u))) << ((rp[k] >> 16) & 63u);
            }
        }
        for (int j = 0; j < PF_BN; ++j) {
            const bool mine = (seen >> j) & 1u;
            if (__ballot(mine) == 0ull) continue;
            const int r = blk * PF_BN + j;                  // (a key that is seen: within the tensor)
            const size_t row = (size_t)(SHARED && !user ? static_cast<const int32_t *>(table)[LOCAL ? own * PF_BN + j : r] : r) * 256;
            const h8 *kp = reinterpret_cast<const h8 *>((user ? Ku : Kf) + row);
            float x = 0.0f;
#pragma unroll
            for (int s = 0; s < 8; ++s) x = dot8(kp[2 * s + g], bq[s], x);
            const float p = (float)(_Float16)__builtin_amdgcn_exp2f(fmaf(cross32_sum(x), c2, mneg));
            const h4 *vp = reinterpret_cast<const h4 *>((user ? Vu : Vf) + row);
            if (mine) {
#pragma unroll
                for (int i8 = 0; i8 < 16; ++i8) {
                    const h4 v = vp[2 * i8 + g];
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[i8][k] = fmaf(p, (float)v[k], o[i8][k]);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (n_split > 1)
            *reinterpret_cast<f4 *>(static_cast<float *>(dst) + 8 * i + 4 * g) = o[i];
        else
            *reinterpret_cast<h4 *>(static_cast<_Float16 *>(dst) + 8 * i + 4 * g) = h4{(_Float16)(o[i][0] * scale), (_Float16)(o[i][1] * scale),
                                                                                      (_Float16)(o[i][2] * scale), (_Float16)(o[i][3] * scale)};
}

// ---- one kept set: shares in proportion ---------------------------------------------------------------------------------
// Heads keep different numbers of keys: with as many shares for every unit the launch ends with the unit that keeps most (8 heads x 512
// tokens x 262144 keys, 16384 clusters: 7 to 23 blocks a workgroup).  So the launch's shares are dealt to the units by their numbers of
// blocks, one each and the rest in proportion, which every wave works out by itself from the counts, a unit per lane.
struct PfDealt {
    int unit, first, n;                                     // the unit, its first share and its number of shares
};
__device__ __forceinline__ PfDealt pf_deal(const PfDeal &deal, int piece, const int32_t *__restrict__ blk_info, int bm, int B, int H,
                                           int L, int Lq, int U, int causal_user)
{
    const int lane = threadIdx.x & 63, u = min(lane, deal.units - 1), nqb = (Lq + bm - 1) / bm;
    const int h = u / (nqb * B), b = (u / nqb) % B, q_end = u % nqb * bm + bm;
    const int kept = max(min(blk_info[2 * ((size_t)b * H + h) + 1], L), 0), seen = causal_user ? min(U, q_end) : U;
    const int blocks = lane < deal.units ? (kept + PF_BN - 1) / PF_BN + (seen + PF_BN - 1) / PF_BN : 0;
    const int incl = wave_inclusive_scan(blocks, lane), all = __builtin_amdgcn_readlane(incl, 63);
    // shares up to and with the lane's unit: one a unit, and the others by the blocks so far (1 of 1 for the last unit)
    const float spare = (float)(deal.shares - deal.units), part = all > 0 ? (float)incl / (float)all : (float)(u + 1) / (float)deal.units;
    const int end = lane < deal.units ? u + 1 + (int)(part * spare + 0.5f) : deal.shares;
    const int before = __builtin_popcountll(__ballot(lane < deal.units && end <= piece));   // units that end in front of this share
    PfDealt d;
    d.unit = before;
    d.first = before > 0 ? __builtin_amdgcn_readlane(end, before - 1) : 0;
    d.n = __builtin_amdgcn_readlane(end, before) - d.first;
    return d;
}

// ---- the kept set made by the attention launch ----------------------------------------------------------------------------
// (mean_row_select.)  Bound by a chain of one round of loads (the clusters' sizes, offsets and up to eight parts of their scores
// together; a further round for every eight parts more, and two in front for candidates, their number and their ids) and three barriers,
// about 3 us of the launch's prologue; the rows' searches run in parallel, a few per thread.
// Rows of the keys of a share's n_list fixed blocks, split, split + n_split, ... of the list of kept keys: every key finds its cluster
// among the records of mean_row_select.  (Behind the last key: that key again.)
template <int PF_WAVES, int MAX_C>
__device__ __forceinline__ void pf_share_rows(const int *s, int32_t *s_idx, int n_list, int split, int n_split, int n_fixed, int L)
{
    const int *s_pos = s, *s_first = s + MAX_C;
    const int kept = s[2 * MAX_C];
    for (int i = threadIdx.x; i < n_list * PF_BN; i += 64 * PF_WAVES) {
        const int j = min((split + (i >> 6) * n_split) * PF_BN + (i & 63), n_fixed - 1);
        int c = 0;
#pragma unroll
        for (int step = MAX_C / 2; step > 0; step >>= 1)
            if (c + step < kept && s_pos[c + step] <= j) c += step;
        s_idx[i] = min(max(s_first[c] + j - s_pos[c], 0), L - 1);   // (malformed offsets stay in the tensor)
    }
}

// SHARED: table is the key-row list [B*H, L] and blk_info the per-row (records, kept keys) headers; keep_mask is not
// used.  Otherwise table / rows / blk_info are the block table (block_table_kernel).
// SELECT (with SHARED): the kept set is made here, from the parts of the averaged scores (what mean_select_kernel does in a launch of
// its own otherwise): every workgroup adds up its head's scores and decides all of its clusters, and the rows of its share's keys go to
// a list in LDS.  The (sequence, head)'s first workgroup writes the mask and the count.  SELECTS: 1 of all clusters, 2 of the row's
// candidates, 0 not.
template <bool SHARED, int PF_WAVES, int SELECTS>
__global__ __launch_bounds__(64 * PF_WAVES, 8 / PF_WAVES) void prefill_attn_kernel(
    const _Float16 *__restrict__ q, const _Float16 *__restrict__ Kf, const _Float16 *__restrict__ Vf,
    const _Float16 *__restrict__ Ku, const _Float16 *__restrict__ Vu, const uint32_t *__restrict__ keep_mask,
    const uint32_t *__restrict__ table, const uint32_t *__restrict__ rows, const int32_t *__restrict__ blk_info,
    _Float16 *__restrict__ out, float *__restrict__ lse, float *__restrict__ partials, int n_split, int B, int H, int L,
    int C, int Lq, int U, int causal_user, float sm_scale, PfSelect sel, PfDeal deal)
{
    constexpr bool SELECT = SELECTS != 0;
    static_assert(SHARED || !SELECT, "one kept set");
    constexpr int SEL_C = pf_select_max_c(PF_WAVES, SELECTS == 2);
    constexpr int PF_BM = pf_bm(PF_WAVES), PF_THREADS = 64 * PF_WAVES;
    constexpr int PF_RP = PF_THREADS / 16;                  // rows of a key block the workgroup moves per pass (16 lanes per row)
    constexpr int PF_NP = PF_BN / PF_RP;                    // passes per block
    static_assert(PF_RP % 16 == 0, "the staging swizzles take the row modulo 16 from the thread alone");
    constexpr int NB = pf_bufs(SHARED, PF_WAVES), LV = NB / 2, LK = LV + 1;   // iteration it fetches V of block it + LV, K of block it + LK
    __shared__ __align__(16) unsigned char stage[2 * NB * PF_TILE];   // NB tiles of K, then NB tiles of V
    __shared__ __align__(16) uint32_t s_tab[SHARED ? 1 : PF_TABS * PF_ROW_WORDS];
    __shared__ uint16_t s_list[SHARED ? 1 : PF_LIST_CAP];   // the fixed blocks this workgroup walks
    __shared__ int s_wc[PF_WAVES], s_act[PF_WAVES];
    __shared__ int s_info[SHARED ? 1 : 64];                 // table entries of the first listed blocks
    __shared__ uint8_t s_need[SHARED ? 1 : PF_LIST_CAP];    // bit v: wave v has a query that kept a key of the listed block
    __shared__ __align__(16) uint32_t s_mw[SHARED ? 1 : PF_WAVES][NB][64];   // mask words of a wave's queries for the blocks at hand (sparse walk)
    __shared__ int32_t s_idx[SELECT ? pf_select_blocks(PF_WAVES) * PF_BN : 1];   // rows of the share's fixed blocks
    __shared__ __align__(16) float s_hide[16 * 4];          // entry n: the start values of four scores whose visibility bits are n

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, g = lane >> 5, l16 = lane & 15;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    if (tid < 64) s_hide[tid] = ((tid >> 2) >> (tid & 3)) & 1 ? 0.0f : SQ_NEG_INF;   // (read behind the barriers below)
    // Workgroup -> (head, sequence, query block, share).  Workgroups are dealt to the 8 XCDs round-robin by their
    // linear id; units that share a head (and so stream the same K/V) are made to land on the same XCD, so
    // one L2 fetches a head's keys once for all of its query blocks.
    const int nqb = (Lq + PF_BM - 1) / PF_BM;
    const int per_xcd = gridDim.x >> 3;                     // grid is a multiple of 8
    const int piece = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (piece >= nqb * B * H * n_split) return;
    // With few (head, query block) units the key blocks of a unit are dealt to n_split workgroups: blocks split,
    // split + n_split, ... (interleaved, so that a run of blocks nobody kept or the causal end of the user keys is shared
    // out evenly).
    int unit = piece / n_split, split = piece - unit * n_split, share0 = 0;   // share0: shares of the units in front (PfDeal)
    if constexpr (SHARED && !SELECT)
        if (deal.units) {                                   // shares in proportion to the units' blocks
            const PfDealt d = pf_deal(deal, piece, blk_info, PF_BM, B, H, L, Lq, U, causal_user);
            unit = d.unit;
            share0 = d.first;
            split = piece - d.first;
            n_split = d.n;
            if (split == 0 && tid == 0) deal.dealt[unit] = int2{d.first, d.n};
        }
    const int h = unit / (nqb * B), b = (unit / nqb) % B;
    const int q0 = (unit % nqb) * PF_BM;                    // first query of the workgroup
    const int W = (C + 31) >> 5;
    const size_t row0 = ((size_t)b * H + h) * Lq;           // query-row index of query 0 of this (b, h)
    const float c2 = sm_scale * 1.44269504088896341f;       // exp(sm_scale * s) = exp2(c2 * s)

    // This lane's query column (a column past the end repeats the last query and is not stored).
    const int q0w = q0 + wave_u * 32, nq = q0w + col, nqc = min(nq, Lq - 1);
    const bool wave_on = q0w < Lq;                          // (wave-uniform)
    h8 bq[8];                                               // B operand of S^T = K Q^T
    {
        const h8 *qp = reinterpret_cast<const h8 *>(q + (row0 + nqc) * D);
#pragma unroll
        for (int s = 0; s < 8; ++s) bq[s] = qp[s * 2 + g];
    }
    float m_ref = SQ_NEG_INF, m_lim = SQ_NEG_INF, mneg = 0.0f, l_run = 0.0f;
    f16v o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;

    const char *Kfh = reinterpret_cast<const char *>(Kf + (size_t)h * L * D), *Vfh = reinterpret_cast<const char *>(Vf + (size_t)h * L * D);
    const char *Kuh = reinterpret_cast<const char *>(Ku + ((size_t)b * H + h) * (size_t)U * D);
    const char *Vuh = reinterpret_cast<const char *>(Vu + ((size_t)b * H + h) * (size_t)U * D);
    // keys of the fixed context this (sequence, head) walks: all of them, or the kept ones through the row list
    int n_fixed = L;
    if constexpr (SELECT)
        n_fixed = min(mean_row_select<PF_WAVES, SEL_C, false, SELECTS == 2>(sel, (size_t)b * H + h, h, C, Lq, unit % nqb == 0 && split == 0,
                                                                            reinterpret_cast<int *>(stage)), L);
    else if constexpr (SHARED)
        n_fixed = min(blk_info[2 * ((size_t)b * H + h) + 1], L);
    const int32_t *idx_bh = reinterpret_cast<const int32_t *>(table) + ((size_t)b * H + h) * (size_t)L;   // SHARED without SELECT only
    const int nblk_fixed = (n_fixed + PF_BN - 1) / PF_BN;
    // Causal user block: queries of this workgroup see user keys 0 .. min(U, q0 + BM) - 1 at most.
    const int u_vis = causal_user ? min(U, q0 + PF_BM) : U;
    const int nblk_user = (u_vis + PF_BN - 1) / PF_BN;
    const int nblk_all = (L + PF_BN - 1) / PF_BN;
    const int32_t *binfo = blk_info + (size_t)h * nblk_all;
    const uint32_t *mrow = keep_mask + (row0 + nqc) * W;    // mask row of this lane's query

    // ---- staging -----------------------------------------------------------------------------------------------------------
    // This thread's pieces of a 64-key block: piece i = key i*PF_RP + tid/16 (rows of 256 B), LDS slot tid%16 of that
    // row, i.e. the 16-byte chunk (tid%16) ^ swz(row) of the row in memory; row % 16 = (tid/16) % 16 for every piece.
    const int trow = tid >> 4;
    const uint32_t k_ch = (uint32_t)((tid & 15) ^ pf_k_swz(trow)) * 16u, v_ch = (uint32_t)((tid & 15) ^ pf_v_swz(trow)) * 16u;
    const uint32_t k_at = (uint32_t)trow * 256u + k_ch, v_at = (uint32_t)trow * 256u + v_ch;
    // Where a block's rows are: base addresses and `end`, 16 bytes before the end of its rows (contiguous rows).
    struct Aim {
        const char *k, *v;
        uint32_t end;
    };
    auto aim_at = [&](int e) PF_INLINE {
        const bool user = e < 0;
        const int j0 = (e & 0x7fffffff) * PF_BN;
        const size_t at = SHARED && !user ? 0 : (size_t)j0 * 256;
        return Aim{(user ? Kuh : Kfh) + at, (user ? Vuh : Vfh) + at, (uint32_t)min((user ? U : L) - j0, PF_BN) * 256u - 16u};
    };
    // SHARED: the gathered rows of this thread's pieces (for a user block the list is not used).
    struct Rows {
        int r[SHARED ? PF_NP : 1];
    };
    auto rows_of = [&](int e) PF_INLINE {
        Rows x{};
        if constexpr (SHARED) {
            const int j0 = e < 0 ? 0 : e * PF_BN, last = max(n_fixed - 1, 0);
#pragma unroll
            for (int k = 0; k < PF_NP; ++k) x.r[k] = idx_bh[min(j0 + k * PF_RP + trow, last)];
        }
        return x;
    };
    typedef __attribute__((address_space(3))) void *lptr_t;
    auto lds_at = [&](const void *p) PF_INLINE { return __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lptr_t)p); };
    // Written as instructions: through the builtin the compiler may make a read of the CURRENT buffer wait for these
    // loads into the OTHER buffer.  The waves wait for their own loads themselves before the barrier that publishes a block.
    // Contiguous rows: rows past the end of the tensor read some chunk in front of it (what lands there is hidden).
    const uint32_t lds_w = lds_at(stage) + (uint32_t)wave_u * 1024u;      // a wave's four rows of a pass: 1 KB, lane l at byte 16 l
    auto fetch_piece = [&](int i, const char *base, uint32_t end, bool gathered, const Rows &rw, uint32_t at, uint32_t ch, uint32_t tile) PF_INLINE {
        uint32_t off = min(at + (uint32_t)i * (PF_RP * 256u), end);
        if constexpr (SHARED) off = gathered ? (uint32_t)rw.r[i] * 256u + ch : off;
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" ::"s"(lds_w),
                     "i"(tile + (uint32_t)i * (PF_RP * 256u)), "v"(off), "s"(base) : "m0", "scc");
    };
    constexpr uint32_t V_AT = NB * PF_TILE;                 // byte offset of the V tiles
    auto loads_landed = [&]() PF_INLINE { __builtin_amdgcn_s_waitcnt(0x0f70); };   // vmcnt(0)

    // ---- the blocks of this share: fixed blocks (masked form: those in which a query of the workgroup kept a cluster, with the
    // waves that need them; nobody's blocks are neither fetched nor staged), then user blocks -------------------------------
    int n_list = (max(nblk_fixed - split, 0) + n_split - 1) / n_split;
    const bool listed = !SHARED && n_list <= PF_LIST_CAP;
    // Masked form: the first blocks of the share are rarely left out, so their tiles are requested before the list is known: they land
    // with the masks instead of a round trip after the list.  With that, the blocks' table entries requested in front of the unions and
    // the first ones kept beside the list, whole steps, us: 16 heads x 200 tokens x 5000 keys 40.2 -> 39.1, 32 x 40 x 8000 42.5 -> 41.8,
    // 4 x 100 x 16000 32.7 -> 31.8, 32 x 1024 x 32768 the same.  Of fewer queries than a wave holds many blocks are left out where a
    // per cent or so of the keys is kept, and the list waits for tiles in vain: 8 x 16 x 100000, 1/100 kept, 72.4 without, 75.0 with
    // them, 8 x 3 x 100000, 1/20 68.1 / 70.6, one head x 1 x 500000, 1/500 52.0 / 54.1; 16 x 20 x 5000, 0.15 27.0 / 26.5.
    const bool ahead = !SHARED && n_list >= LK && Lq >= 32;
    if (ahead)
#pragma unroll
        for (int b = 0; b < LK; ++b) {
            const Aim aim = aim_at(split + b * n_split);
#pragma unroll
            for (int i = 0; i < PF_NP; ++i) {
                fetch_piece(i, aim.k, aim.end, false, Rows{}, k_at, k_ch, b * PF_TILE);
                if (b < LV) fetch_piece(i, aim.v, aim.end, false, Rows{}, v_at, v_ch, V_AT + b * PF_TILE);
            }
        }
    if constexpr (SELECT) {
        static_assert(sizeof(stage) >= mean_row_cand_words(SEL_C) * sizeof(int), "the records lie where the tiles will be");
        pf_share_rows<PF_WAVES, SEL_C>(reinterpret_cast<const int *>(stage), s_idx, n_list, split, n_split, n_fixed, L);
        __syncthreads();                                    // (the records lie where the tiles will be)
    }
    bool sparse = false;
    if (listed) {
        // per wave: OR of the keep masks of its queries, in a tile that the first fetches leave alone
        uint32_t *s_um = reinterpret_cast<uint32_t *>(stage + (NB == 4 ? LK * PF_TILE : V_AT + LV * PF_TILE));
        static_assert(NB == 4 ? LK < NB : LV < NB, "");
        static_assert(PF_TILE >= PF_WAVES * PF_UMASK_WORDS * 4, "the unions fit a tile");
        int bi = tid < n_list ? binfo[split + tid * n_split] : 0;   // (requested in front of the unions' round trip)
        pf_union_masks(s_um, keep_mask, row0, q0, PF_WAVES, Lq, W, tid, PF_THREADS);
        int base = 0, active = 0;                           // blocks listed; (wave, block) pairs with a kept key, of this thread's blocks
        for (int i0 = 0; i0 < n_list; i0 += PF_THREADS) {   // in order: a ballot per wave, the waves' counts in LDS
            const int bb = split + (i0 + tid) * n_split;
            int waves = 0;
            if (i0 > 0) bi = i0 + tid < n_list ? binfo[bb] : 0;
            if (i0 + tid < n_list) {
                for (int v = 0; v < PF_WAVES; ++v) waves |= (int)pf_block_needed(bi, s_um + v * W, W) << v;
            }
            const bool need = waves != 0;
            active += __popc(waves);
            const unsigned long long bal = __ballot(need);
            if (lane == 0) s_wc[wave] = __popcll(bal);
            __syncthreads();
            int before = 0, total = 0;
#pragma unroll
            for (int w = 0; w < PF_WAVES; ++w) {
                if (w < wave) before += s_wc[w];
                total += s_wc[w];
            }
            if (need) {
                const int at = base + before + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
                s_list[at] = (uint16_t)bb;
                s_need[at] = (uint8_t)waves;
                if (at < 64) s_info[at] = bi;
            }
            base += total;
            __syncthreads();
        }
        n_list = __builtin_amdgcn_readfirstlane(base);
        const int act = (int)wave_sum((float)active);
        if (lane == 0) s_act[wave] = act;
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int w = 0; w < PF_WAVES; ++w) all += s_act[w];
        all = __builtin_amdgcn_readfirstlane(all);
        sparse = all * PF_SPARSE_DEN < n_list * min(PF_WAVES, (Lq - q0 + 31) >> 5) * PF_SPARSE_NUM;   // (of the waves with queries)
    }
    const int half = NB == 4 && sparse ? (n_list + 1) >> 1 : 0;   // (position 2 i + 1 is listed half a list behind position 2 i)
    const int u_first = (split + n_split - nblk_fixed % n_split) % n_split;   // first user block of the share
    const int n_mine = n_list + (max(nblk_user - u_first, 0) + n_split - 1) / n_split;
    // The walk's next entries, one per lane: lane i holds position t_base + i (past the end: the last one again) as block | user
    // flag << 31, and a fixed block's table entry.  Read with v_readlane, refilled every few dozen blocks: scalar values that
    // cost one instruction each.
    int t_base = 0, t_ent = 0, t_info = 0, t_need = 0;
    auto fill_entries = [&](int base) PF_INLINE {
        t_base = base;
        const int i = min(base + lane, n_mine - 1);
        const bool user = i >= n_list;
        const int li = half ? (i >> 1) + (i & 1) * half : i;
        const int blk = user ? u_first + (i - n_list) * n_split : listed ? (int)s_list[li] : split + i * n_split;
        t_ent = user ? blk | (int)0x80000000 : blk;
        if (!SHARED) {
            // (the first entries' from LDS, behind the list; a user block's is not looked at)
            if (base == 0 && listed && !half) t_info = user ? 0 : s_info[li & 63];
            else t_info = binfo[user ? 0 : blk];
            // (waited for here: left pending, it makes the compiler wait in every block, for the tiles on their way as well)
            asm volatile("" : "+v"(t_info));
            t_need = user || !listed ? 0xff : s_need[li];
        }
    };
    auto ent = [&](int i) PF_INLINE { return __builtin_amdgcn_readlane(t_ent, i - t_base); };
    auto inf = [&](int i) PF_INLINE { return __builtin_amdgcn_readlane(t_info, i - t_base); };
    constexpr int T_KEEP = 56;                              // entries used of a fill: the loop looks up to seven ahead

    auto rows_at = [&](int i) PF_INLINE {                   // of the block at position i
        if constexpr (SELECT) {
            Rows x{};
#pragma unroll
            for (int k = 0; k < PF_NP; ++k) x.r[k] = s_idx[min(i, max(n_list - 1, 0)) * PF_BN + k * PF_RP + trow];
            return x;
        } else
            return rows_of(ent(i));
    };

    // Masked form: what decides the visible keys travels ahead of the block: its table row to LDS (one wave fetches it), and
    // the two mask words of this lane's query that hold the block's window of clusters (loaded when the window moves to
    // another word, every few blocks).
    auto fetch_tab = [&](int pos, int e) PF_INLINE {
        if (SHARED || wave_u != 0) return;
        const uint32_t *p = rows + ((size_t)h * nblk_all + (e < 0 ? 0 : e)) * PF_ROW_WORDS;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_at(s_tab) + (uint32_t)(pos & (PF_TABS - 1)) * (PF_ROW_WORDS * 4)),
                     "v"(lane * 4), "s"(p) : "m0");
    };
    uint32_t mw_lo = 0u, mw_hi = 0u;                        // (pipelined walk)
    int mw_at = -1;
    auto fetch_words = [&](int info) PF_INLINE {
        if (SHARED) return;
        const int w0 = (info & 0xffff) >> 5;
        if (w0 != mw_at) {
            mw_at = w0;
            mw_lo = mrow[min(w0, W - 1)];
            mw_hi = w0 + 1 < W ? mrow[w0 + 1] : 0u;
        }
    };
    // Keys of the block with entry e (table entry info; pos: its walk position) that this lane's query sees, as the accumulators
    // hold them: bit 8 a + i of w[t] = key 32 t + 8 a + 4 g + i (i < 4).
    auto visible_edge = [&](int e, uint32_t (&w)[2]) PF_INLINE {
        // user keys: those at or before the query (causal); one kept set: all but the slots past the kept keys
        const int n = (e >= 0 ? n_fixed : causal_user ? min(U, nqc + 1) : U) - (e & 0x7fffffff) * PF_BN;
        const unsigned long long m = n >= 64 ? ~0ull : (1ull << max(n, 0)) - 1ull;
        w[0] = (uint32_t)(m >> (4 * g)) & 0x0f0f0f0fu;
        w[1] = (uint32_t)(m >> 32 >> (4 * g)) & 0x0f0f0f0fu;
    };
    auto visible_runs = [&](int e, int info, uint32_t (&w)[2]) PF_INLINE {       // every run's bit from the mask itself
        const uint32_t *rp = table + ((size_t)h * nblk_all + e) * PF_BN;
        w[0] = w[1] = 0u;
        for (int i = 0; i < ((info >> 21) & 127); ++i) {
            const uint32_t r = __builtin_amdgcn_readfirstlane(rp[i]), c = r & 0xffffu;
            const unsigned long long ks = (~0ull >> (63 - (int)((r >> 22) & 63u))) << ((r >> 16) & 63u);
            const uint32_t on = 0u - ((mrow[c >> 5] >> (c & 31u)) & 1u);
            w[0] |= on & (uint32_t)(ks >> (4 * g)) & 0x0f0f0f0fu;
            w[1] |= on & (uint32_t)(ks >> 32 >> (4 * g)) & 0x0f0f0f0fu;
        }
    };
    auto visible = [&](int pos, int e, int info, uint32_t wl, uint32_t wh, uint32_t (&w)[2]) PF_INLINE {
        if (SHARED || e < 0) return visible_edge(e, w);
        const int n = (info >> 21) & 127, first = info & 0xffff;
        if (info < 0 || n > PF_ROW_RUNS) return visible_runs(e, info, w);   // more than 31 cluster ids, or many runs
        // bit (cluster - first cluster of the block) of the query's window, spread over the keys of its run
        const uint32_t qb = __builtin_amdgcn_alignbit(wh, wl, (uint32_t)first & 31u) & 0x7fffffffu;
        const uint32_t *row = s_tab + (pos & (PF_TABS - 1)) * PF_ROW_WORDS;
        w[0] = w[1] = 0u;
        auto group = [&](int k) PF_INLINE {
            const uint4 rel = *reinterpret_cast<const uint4 *>(row + k * PF_ROW_GROUP);
            const uint4 k0 = *reinterpret_cast<const uint4 *>(row + k * PF_ROW_GROUP + 4 + 8 * g);
            const uint4 k1 = *reinterpret_cast<const uint4 *>(row + k * PF_ROW_GROUP + 8 + 8 * g);
            auto add = [&](uint32_t r, uint32_t a, uint32_t b) PF_INLINE {
                const uint32_t on = (uint32_t)__builtin_amdgcn_sbfe((int)qb, r, 1u);
                w[0] |= on & a;
                w[1] |= on & b;
            };
            add(rel.x, k0.x, k1.x);
            add(rel.y, k0.y, k1.y);
            add(rel.z, k0.z, k1.z);
            add(rel.w, k0.w, k1.w);
        };
        group(0);
        if (n > 4) {
            group(1);
            group(2);
        }
    };

    // Operand addresses in LDS, of the first stage's tiles (the swizzles depend on the lane alone); hidden from the compiler,
    // which would otherwise add their two parts again in front of every read.
    uint32_t k_lds[8], v_lds[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        k_lds[i] = (uint32_t)(size_t)(lptr_t)stage + (uint32_t)(col * D + ((2 * i + g) ^ pf_k_swz(l16)) * 8) * 2u;
        asm volatile("" : "+v"(k_lds[i]));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 4 * g + (l16 >> 2), chunk = i * 4 + 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);
        v_lds[i] = (uint32_t)(size_t)(lptr_t)stage + V_AT + (uint32_t)(row * D + (chunk ^ pf_v_swz(row)) * 8 + (l16 & 1) * 4) * 2u;
        asm volatile("" : "+v"(v_lds[i]));
    }
    typedef __attribute__((address_space(3))) const h8 *lds_h8_t;
    typedef __attribute__((address_space(3))) tr_h4 *lds_tr_t;
    auto k_operand = [&](uint32_t st, int m) PF_INLINE {              // product m: keys (m & 1) * 32 .. + 31, dimensions 16 (m >> 1) .. + 15
        return *(lds_h8_t)(k_lds[m >> 1] + st + (uint32_t)(m & 1) * (32u * D * 2u));
    };
    auto v_operand = [&](uint32_t st, int m) PF_INLINE {              // product m: keys 16 (m >> 2) .. + 15, dimensions 32 (m & 3) .. + 31
        const uint32_t at = v_lds[m & 3] + st + (uint32_t)(m >> 2) * (16u * D * 2u);
        const h4 a0 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_tr_t)at));
        const h4 a1 = __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_tr_t)(at + 8u * D * 2u)));
        return h8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
    };
    // A block's score products start from 0 for a pair that is visible and -inf for one that is hidden: masks cost no vector
    // arithmetic, four start values come with one LDS read.  Group gi = 4 t + a: keys 32 t + 8 a + 4 g + (0..3).
    auto start_group = [&](f16v (&sa)[2], const uint32_t (&w)[2], int gi) PF_INLINE {
        const int t = gi >> 2, a = gi & 3;
        const f4 v = *reinterpret_cast<const f4 *>(s_hide + ((w[t] >> (8 * a)) & 0xffu) * 4);
#pragma unroll
        for (int k = 0; k < 4; ++k) sa[t][4 * a + k] = v[k];
    };
    auto max_pair = [&](float mx, const f16v (&sa)[2], int i) PF_INLINE {    // (propagates NaN: see new_max)
        const int t = i >> 3, r = 2 * (i & 7);
        return __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, sa[t][r]), sa[t][r + 1]);
    };
    // The reference maximum moves only when a score passes it by 2^8 (probabilities then stay below 2^8, far inside
    // fp16's range, at the same relative rounding): the output is rarely rescaled.  A hidden key with an infinite or NaN
    // component makes its score NaN instead of -inf: such a block's hidden scores are set again here (w0, w1: its visible
    // keys), and the maximum is then taken without regard to NaN.
    auto new_max = [&](float mx, f16v (&sa)[2], uint32_t w0, uint32_t w1) PF_INLINE {
        if (__ballot(!(mx <= m_lim)) != 0ull) {
            if (__ballot(mx != mx) != 0ull) {
                mx = SQ_NEG_INF;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        sa[t][r] = ((t ? w1 : w0) >> (8 * (r >> 2) + (r & 3))) & 1u ? sa[t][r] : SQ_NEG_INF;
                        mx = fmaxf(mx, sa[t][r]);
                    }
            }
            const float m_new = fmaxf(m_ref, cross32_max(mx));
            const float alpha = m_new == m_ref ? 1.0f : __builtin_amdgcn_exp2f((m_ref - m_new) * c2);
            m_ref = m_new;
            m_lim = m_new + 8.0f / c2;
            mneg = m_new == SQ_NEG_INF ? 0.0f : -m_new * c2;       // nothing seen yet: exp2(-inf) = 0
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
        }
    };

    if (!SHARED && sparse && n_mine > 0) {                  // the sparse walk
        fill_entries(0);
        // What the block at position pos needs, behind the barrier that ends the pair before it (NB = 2: the block before it): its
        // tiles, its table row and, for a wave that needs the block, the two words of its queries' masks that hold the block's window
        // of clusters (lane = query + 32 word).
        const uint32_t *mw_base = keep_mask + (row0 + min(q0w, Lq - 1)) * W;
        const uint32_t mw_row = (uint32_t)(nqc - min(q0w, Lq - 1)) * (uint32_t)W;
        auto needed = [&](int pos) PF_INLINE { return wave_on && ((__builtin_amdgcn_readlane(t_need, pos - t_base) >> wave_u) & 1); };
        auto fetch_window = [&](int pos, int slot) PF_INLINE {
            const int w0 = (inf(pos) & 0xffff) >> 5;        // (a window that begins in the last word needs no second one)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_at(&s_mw[wave_u][slot][0])),
                         "v"((mw_row + (uint32_t)min(w0 + g, W - 1)) * 4u), "s"(mw_base) : "m0");
        };
        auto fetch_at = [&](int pos, auto tile) PF_INLINE {
            const int e = ent(pos);
            const Aim aim = aim_at(e);
#pragma unroll
            for (int i = 0; i < PF_NP; ++i) {
                fetch_piece(i, aim.k, aim.end, false, Rows{}, k_at, k_ch, tile * PF_TILE);
                fetch_piece(i, aim.v, aim.end, false, Rows{}, v_at, v_ch, V_AT + tile * PF_TILE);
            }
            fetch_tab(pos, e);
            if (needed(pos)) fetch_window(pos, tile);
        };
        if (ahead) loads_landed();                          // (the same tiles are fetched, of other blocks)
        fetch_at(0, std::integral_constant<int, 0>{});
        if (NB == 4) fetch_at(1, std::integral_constant<int, 1>{});
        loads_landed();
        __syncthreads();
        auto step = [&](int it, auto par) PF_INLINE {
            constexpr uint32_t at = par * PF_TILE;
            if (NB == 2) fetch_at(it + 1, std::integral_constant<int, (par + 1) % NB>{});
            else if (par % 2 == 0) {                        // both of the next pair: its loads have this pair's time to land
                fetch_at(it + 2, std::integral_constant<int, (par + 2) % NB>{});
                fetch_at(it + 3, std::integral_constant<int, (par + 3) % NB>{});
            }
            uint32_t w[2] = {0u, 0u};
            if (needed(it)) visible(it, ent(it), inf(it), s_mw[wave_u][par][col], s_mw[wave_u][par][32 + col], w);
            if (__ballot((w[0] | w[1]) != 0u) != 0ull) {
                f16v sc[2];
#pragma unroll
                for (int gi = 0; gi < 8; ++gi) start_group(sc, w, gi);
#pragma unroll
                for (int m = 0; m < 16; ++m)
                    sc[m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(k_operand(at, m), bq[m >> 1], sc[m & 1], 0, 0, 0);
                float mx = SQ_NEG_INF, ps0 = 0.0f, ps1 = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = max_pair(mx, sc, i);
                new_max(mx, sc, w[0], w[1]);
                h8 bp[4];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int t = i >> 3, r = 2 * (i & 7);
                    const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[t][r], c2, mneg));
                    const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[t][r + 1], c2, mneg));
                    ps0 += p0;
                    ps1 += p1;
                    bp[2 * t + (r >> 3)][r & 7] = (_Float16)p0;
                    bp[2 * t + (r >> 3)][(r & 7) + 1] = (_Float16)p1;
                }
                l_run += ps0 + ps1;
#pragma unroll
                for (int m = 0; m < 16; ++m)
                    o[m & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v_operand(at, m), bp[m >> 2], o[m & 3], 0, 0, 0);
            }
            if (it + 1 - t_base >= T_KEEP) fill_entries(it + 1);
            if (NB == 2 || (par & 1)) {
                loads_landed();
                __syncthreads();
            }
        };
        for (int it = 0; it < n_mine; it += NB) {
            step(it, std::integral_constant<int, 0>{});
            if (it + 1 < n_mine) step(it + 1, std::integral_constant<int, 1>{});
            if constexpr (NB == 4) {
                if (it + 2 < n_mine) step(it + 2, std::integral_constant<int, 2>{});
                if (it + 3 < n_mine) step(it + 3, std::integral_constant<int, 3>{});
            }
        }
    } else if (n_mine > 0) {                                // (no kept key and no user key: nothing to do)
        fill_entries(0);
        f16v s_cur[2], s_nxt[2];
        uint32_t vis0 = 0u, vis1 = 0u;                      // visible keys of the block whose start values were made last
        uint2 w2{}, w3{};                                   // mask words of blocks it + 2, it + 3
        bool any_cur = true, any_nxt = true;                // does this wave see a key of block it, it + 1?
        // Start values of the scores of the block at position i; nothing visible past the end of the walk.
        auto start_scores = [&](f16v (&sa)[2], int i, uint2 words) PF_INLINE {
            uint32_t w[2] = {0u, 0u};
            if (i < n_mine) visible(i, ent(i), inf(i), words.x, words.y, w);
            vis0 = w[0];
            vis1 = w[1];
#pragma unroll
            for (int gi = 0; gi < 8; ++gi) start_group(sa, w, gi);
            return __ballot((w[0] | w[1]) != 0u) != 0ull;
        };
        auto words_of = [&](int i) PF_INLINE {
            fetch_words(inf(i));
            return uint2{mw_lo, mw_hi};
        };
        Aim aim_v{};                                        // of block it + LV (computed with its K, one iteration before)
        Rows rv = rows_at(LV), rk = rows_at(LK), rk1 = rows_at(LK + 1);   // blocks it + LV, it + LK, it + LK + 1
        bool there = ahead;                                 // are the tiles that were requested those of the list's first blocks?
#pragma unroll
        for (int b = 0; b < LK; ++b) there = there && ent(b) == split + b * n_split;
        if (ahead && !there) loads_landed();
#pragma unroll
        for (int b = 0; b < LK; ++b) {
            const int e = ent(b);
            aim_v = aim_at(e);
            if (there) continue;                            // (uniform)
            const Rows r = rows_at(b);
#pragma unroll
            for (int i = 0; i < PF_NP; ++i) {
                fetch_piece(i, aim_v.k, aim_v.end, e >= 0, r, k_at, k_ch, b * PF_TILE);
                if (b < LV) fetch_piece(i, aim_v.v, aim_v.end, e >= 0, r, v_at, v_ch, V_AT + b * PF_TILE);
            }
        }
#pragma unroll
        for (int b = 0; b < PF_TABS; ++b) fetch_tab(b, ent(b));
        const uint2 w0 = words_of(0), w1 = words_of(1);
        w2 = words_of(2);
        w3 = words_of(3);
        loads_landed();
        __syncthreads();
        if (wave_on) {                                      // scores of the first block
            any_cur = start_scores(s_cur, 0, w0);
#pragma unroll
            for (int m = 0; m < 16; ++m)
                s_cur[m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(k_operand(0u, m), bq[m >> 1], s_cur[m & 1], 0, 0, 0);
            float mx = SQ_NEG_INF;
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = max_pair(mx, s_cur, i);
            new_max(mx, s_cur, vis0, vis1);
            any_nxt = start_scores(s_nxt, 1, w1);
        }
        __syncthreads();                                    // K of the first block is read: its buffer may be filled again

        // Iteration it: softmax of block it (scores ready, maximum known), S^T = K Q^T of block it + 1, O^T += V^T P^T of block
        // it, then the maximum of block it + 1 and the start values of block it + 2.  Matrix and vector work are laid out
        // alternating in the instruction stream: 24 products between the 16 pairs of exponentials, 8 between the rest; the
        // scalar work that aims the next loads goes behind the first products.
        // masked: std::bool_constant; false: the blocks up to it + LK are full blocks of kept keys, every pair visible.
        auto walk = [&](int it, auto par, f16v (&sc)[2], f16v (&sn)[2], auto masked) PF_INLINE {
            constexpr bool MASKED = decltype(masked)::value;
            constexpr uint32_t at_v = par * PF_TILE, at_k = (par + 1) % NB * PF_TILE;
            constexpr uint32_t to_v = V_AT + (par + LV) % NB * PF_TILE, to_k = (par + LK) % NB * PF_TILE;
            Aim aim_k{};
            bool gk = true, gv = true;
            Rows rk2{};
            uint2 w4{};
            auto look_ahead = [&]() PF_INLINE {
                const int e = ent(it + LK);
                aim_k = aim_at(e);
                if (MASKED) {
                    gk = e >= 0;
                    gv = ent(it + LV) >= 0;
                }
            };
            auto look_further = [&]() PF_INLINE {
                rk2 = rows_at(it + LK + 2);
                fetch_tab(it + 4, ent(it + 4));
                w4 = words_of(it + 4);
            };
            auto fetch_kv = [&](int x) PF_INLINE {                    // 2 PF_NP pieces; the tiles they fill were read one pass ago or earlier
                if (x & 1) fetch_piece(x >> 1, aim_v.v, aim_v.end, gv, rv, v_at, v_ch, to_v);
                else fetch_piece(x >> 1, aim_k.k, aim_k.end, gk, rk, k_at, k_ch, to_k);
            };
            // A wave that sees no key of the three blocks at hand has nothing to do: hidden scores stay -inf, whatever block they
            // belong to.  (User keys after the wave's queries; runs of blocks that only other waves need.)
            bool any_new = true, on = wave_on;
            if (MASKED && on && !any_cur && !any_nxt) {
                uint32_t w[2] = {0u, 0u};
                if (it + 2 < n_mine) visible(it + 2, ent(it + 2), inf(it + 2), w2.x, w2.y, w);
                any_new = on = __ballot((w[0] | w[1]) != 0u) != 0ull;
            }
            if (on) {
                h8 op[PF_AHEAD];
                auto operand = [&](int m) PF_INLINE { return m < 16 ? k_operand(at_k, m) : v_operand(at_v, m - 16); };
#pragma unroll
                for (int m = 0; m < PF_AHEAD; ++m) op[m] = operand(m);
                h8 bp[4];
                float ps0 = 0.0f, ps1 = 0.0f, mx = SQ_NEG_INF;
                const uint32_t v0 = MASKED ? vis0 : ~0u, v1 = MASKED ? vis1 : ~0u;
                uint32_t w[2] = {0u, 0u};
                __builtin_amdgcn_sched_barrier(0);
                static_for<32>([&](auto ic) PF_INLINE {
                    constexpr int i = ic;
                    if constexpr (i < 16) {                 // two probabilities of block it
                        constexpr int t = i >> 3, r = 2 * (i & 7);
                        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[t][r], c2, mneg));
                        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[t][r + 1], c2, mneg));
                        ps0 += p0;
                        ps1 += p1;
                        bp[2 * t + (r >> 3)][r & 7] = (_Float16)p0;
                        bp[2 * t + (r >> 3)][(r & 7) + 1] = (_Float16)p1;
                        asm volatile("" : "+v"(ps0), "+v"(ps1));   // (the sums stay here, between the products)
                        if constexpr (i == 1) look_ahead();
                        if constexpr (i >= 2 && i < 2 + 2 * PF_NP) fetch_kv(i - 2);
                        if constexpr (i == 11) look_further();
                    } else {                                // two scores of block it + 1, four start values of block it + 2
                        mx = max_pair(mx, sn, i - 16);
                        asm volatile("" : "+v"(mx));
                        if constexpr (MASKED) {
                            if constexpr (i == 16) {
                                if (it + 2 < n_mine) visible(it + 2, ent(it + 2), inf(it + 2), w2.x, w2.y, w);
                                vis0 = w[0];
                                vis1 = w[1];
                                any_new = __ballot((w[0] | w[1]) != 0u) != 0ull;
                            }
                            if constexpr (i & 1) start_group(sc, w, (i - 16) >> 1);
                        }
                    }
                    constexpr int m0 = i < 16 ? 3 * i / 2 : 24 + (i - 16) / 2, m1 = i < 16 ? 3 * (i + 1) / 2 : 24 + (i - 15) / 2;
                    static_for<m1 - m0>([&](auto mc) PF_INLINE {
                        constexpr int m = m0 + mc;
                        const h8 a = op[m % PF_AHEAD];
                        if constexpr (m < 2 && !MASKED) {
                            f16v z;
#pragma unroll
                            for (int r = 0; r < 16; ++r) z[r] = 0.0f;
                            sn[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bq[0], z, 0, 0, 0);
                        } else if constexpr (m < 16)
                            sn[m & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bq[m >> 1], sn[m & 1], 0, 0, 0);
                        else
                            o[m & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bp[(m - 16) >> 2], o[m & 3], 0, 0, 0);
                        if constexpr (m + PF_AHEAD < 32) op[m % PF_AHEAD] = operand(m + PF_AHEAD);
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                l_run += ps0 + ps1;
                new_max(mx, sn, v0, v1);
            } else {
                look_ahead();
#pragma unroll
                for (int x = 0; x < 2 * PF_NP; ++x) fetch_kv(x);
                look_further();
            }
            any_cur = any_nxt;
            any_nxt = any_new;
            aim_v = aim_k;
            rv = rk;
            rk = rk1;
            rk1 = rk2;
            w2 = w3;
            w3 = w4;
            if (it + 1 - t_base >= T_KEEP) fill_entries(it + 1);
            if (NB == 2 || (par & 1)) {
                loads_landed();
                __syncthreads();
            }
        };
        // Unrolled over the LDS buffers: which one is read and which is filled are compile-time constants, so the swizzled
        // operand addresses are loop-invariant plus an immediate.
        int it = 0;
        auto walks = [&](auto masked) PF_INLINE {
            walk(it, std::integral_constant<int, 0>{}, s_cur, s_nxt, masked);
            if (!masked || it + 1 < n_mine) walk(it + 1, std::integral_constant<int, 1>{}, s_nxt, s_cur, masked);
            if constexpr (NB == 4) {
                if (!masked || it + 2 < n_mine) walk(it + 2, std::integral_constant<int, 2>{}, s_cur, s_nxt, masked);
                if (!masked || it + 3 < n_mine) walk(it + 3, std::integral_constant<int, 3>{}, s_nxt, s_cur, masked);
            }
        };
        if constexpr (SHARED) {                             // while the blocks fetched ahead are full blocks of kept keys: no start values
            const int n_full = (max(n_fixed / PF_BN - split, 0) + n_split - 1) / n_split;
            for (; it + NB - 1 + LK < n_full; it += NB) walks(std::false_type{});
            if (it > 0 && wave_on) any_nxt = start_scores(s_nxt, it + 1, uint2{0u, 0u});
        }
        for (; it < n_mine; it += NB) walks(std::true_type{});
    } else if (ahead)
        loads_landed();                                     // (nothing may be on its way to LDS behind the end)

    // ---- values that are not finite ------------------------------------------------------------------------------------------
    // The products of a block multiply the values of keys that a query does not see (and of rows past the end of a tensor) by 0,
    // which is NaN where the value is infinite or NaN.  A query with a NaN in its output (finite inputs cannot cause that) takes it
    // again from the keys it sees alone.
    float top[4];                                           // (the maximum propagates NaN)
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        top[dt] = o[dt][0];
#pragma unroll
        for (int r = 1; r < 15; r += 2) top[dt] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top[dt], o[dt][r]), o[dt][r + 1]);
        top[dt] = __builtin_elementwise_maximum(top[dt], o[dt][15]);
    }
    const float bad = cross32_sum(__builtin_elementwise_maximum(__builtin_elementwise_maximum(top[0], top[1]), __builtin_elementwise_maximum(top[2], top[3])));   // (a query's two lanes hold half of its dimensions each)
    const bool again = bad != bad;

    // ---- normalise and store: lane holds query column nq, dims dt*32 + 8*a + 4*g + (0..3) --------------------------------
    const float lt = cross32_sum(l_run);
    if (nq >= Lq) return;
    const bool empty = !(lt > 0.0f);
    const float inv = empty ? 0.0f : 1.0f / lt;
    _Float16 *orow = out + (row0 + nq) * D;
    const bool dealt = SHARED && !SELECT && deal.units != 0;   // (uniform)
    float *pr = partials + ((dealt ? (size_t)share0 * deal.rows + (size_t)(nq - q0) * n_split : (row0 + nq) * (size_t)n_split) + split) * PART_STRIDE;
    if (n_split > 1) {                                      // this share's (m, l, o) for the merge launch; m in natural units
        if (!again)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    *reinterpret_cast<f4 *>(pr + 4 + dt * 32 + 8 * a + 4 * g) = f4{o[dt][4 * a], o[dt][4 * a + 1], o[dt][4 * a + 2], o[dt][4 * a + 3]};
        if (g == 0) {
            pr[0] = m_ref * sm_scale;
            pr[1] = lt;
        }
    } else {
        if (!again)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    h4 hv;
#pragma unroll
                    for (int v = 0; v < 4; ++v) hv[v] = (_Float16)(o[dt][4 * a + v] * inv);
                    *reinterpret_cast<h4 *>(orow + dt * 32 + 8 * a + 4 * g) = hv;
                }
        if (lse && g == 0) lse[row0 + nq] = empty ? SQ_NEG_INF : m_ref * sm_scale + logf(lt);
    }
    if (again)
        prefill_again<SHARED, SELECT>(q + (row0 + nq) * D, Kfh, Vfh, Kuh, Vuh, mrow,
                              SELECT ? (const void *)s_idx : SHARED ? (const void *)idx_bh : (const void *)(table + (size_t)h * nblk_all * PF_BN), binfo,
                              n_split > 1 ? (void *)(pr + 4) : (void *)orow, split, n_split, n_fixed, U,
                              causal_user ? min(U, nq + 1) : U, c2, mneg, inv);
}

// Merges the n_split partial results of a query row.  GROUPS half waves per row, four dimensions per lane: half wave i takes shares
// i, i + GROUPS, ..., AHEAD of them under way together, with a running maximum, and their results meet in LDS.  Bound by the
// partials' bytes where rows are many (528 per row and share, just written), by one round of loads where they are few.
// Only a row's own shares are folded, each once: a share's sums may be infinite or NaN, and even without weight they would reach
// the result.  So AHEAD is what the shares divide into (ONE: a single round), and a slot that may lie past the end -- the last one,
// and with several rounds any -- holds zeros there, a select per value; the loads are fenced off, between which the compiler puts
// the selects otherwise.
// Traced, a wave per row that found the maximum first / eight shares a round, the last of them taken again to fill it / this kernel:
// 32768 rows x 2 shares 11.7 / 8.2 / 7.8 us, 7992 x 7 7.2 / 6.4 / 5.9, 4096 x 16 8.0 / 7.7 / 7.3; 4096 x 10 6.5 / 5.4, 3000 x 11
// 4.9 / 4.5, 3000 x 17 8.2 / 7.1, 1000 x 24 5.2 / 4.1, 100 x 63 4.0 / 3.9 (the last two of the three).
// DEALT: rows are units times deal.rows positions, and the attention launch named every unit's first share and number of shares.  Only
// the device knows how many: a workgroup, whose rows are of one unit, branches to the form with rounds as even as they go.  (Traced, a
// fixed eight shares a round / this: 16384 rows x 4 shares on average 9.6 / 9.0 us, 5140 x 8 7.9 / 7.1, 4096 x 16 9.1 / 8.8; known on the
// host, without dealing: 6.6, 4.6.)
struct PfMerge {
    PfDeal deal;
    int nqb, B, H, Lq;
};
template <int AHEAD, int GROUPS, bool ONE, bool DEALT>
__global__ __launch_bounds__(256) void prefill_merge_kernel(const float *__restrict__ partials, _Float16 *__restrict__ out,
                                                            float *__restrict__ lse, int n_split, size_t rows, PfMerge mg)
{
    const int half = threadIdx.x >> 5, lane = threadIdx.x & 31, group = half % GROUPS;
    size_t row = (size_t)blockIdx.x * (8 / GROUPS) + half / GROUPS;
    const float *pr = partials + min(row, rows - 1) * (size_t)n_split * PART_STRIDE;
    if constexpr (DEALT) {                                  // (a workgroup's rows are of one unit: deal.rows is a multiple of 8)
        const int first = (int)blockIdx.x * (8 / GROUPS), unit = first / mg.deal.rows;   // (uniform, as all that follows from them)
        const int r0 = first - unit * mg.deal.rows, q0 = unit % mg.nqb * mg.deal.rows, bh = unit / mg.nqb % mg.B * mg.H + unit / (mg.nqb * mg.B);
        const int2 d = mg.deal.dealt[unit];
        n_split = __builtin_amdgcn_readfirstlane(d.y);
        if (n_split == 1 || q0 + r0 >= mg.Lq) return;       // (its only share wrote the outputs; no row of the workgroup is a query)
        const int r = r0 + half / GROUPS;
        pr = partials + ((size_t)d.x * mg.deal.rows + (size_t)r * n_split) * PART_STRIDE;
        rows = (size_t)mg.B * mg.H * mg.Lq;
        row = q0 + r < mg.Lq ? (size_t)bh * mg.Lq + q0 + r : rows;
    }
    float M = SQ_NEG_INF, l = 0.0f;
    f4 o = {0.f, 0.f, 0.f, 0.f};
    auto fold = [&](const auto &m, const auto &n, const auto &v) {
        constexpr int N = (int)std::extent_v<std::remove_reference_t<decltype(m)>>;
        float top = M;
#pragma unroll
        for (int k = 0; k < N; ++k) top = fmaxf(top, m[k]);
        const float old = M == SQ_NEG_INF ? 0.0f : expf(M - top);
        l *= old;
        o *= old;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float w = m[k] == SQ_NEG_INF ? 0.0f : expf(m[k] - top);
            l = fmaf(w, n[k], l);
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] = fmaf(w, v[k][d], o[d]);
        }
        M = top;
    };
    auto take = [&](auto ahead) PF_INLINE {                 // all of the half wave's shares, `ahead` of them in a round
        constexpr int A = ahead;
        for (int s0 = group; ONE ? s0 == group : s0 < n_split; s0 += A * GROUPS) {
            float m[A], n[A];
            f4 v[A];
            constexpr auto full = [](int k) { return ONE && (GROUPS == 1 || k < A - 1); };
#pragma unroll
            for (int k = 0; k < A; ++k) {
                const float *p = pr + (size_t)(full(k) ? s0 + k * GROUPS : min(s0 + k * GROUPS, n_split - 1)) * PART_STRIDE;
                const float2 ml = *reinterpret_cast<const float2 *>(p);
                m[k] = ml.x;
                n[k] = ml.y;
                v[k] = *reinterpret_cast<const f4 *>(p + 4 + 4 * lane);
            }
            __builtin_amdgcn_sched_barrier(0);              // (all of them under way)
#pragma unroll
            for (int k = 0; k < A; ++k) {                   // past the end: zeros, no share's values, which may be infinite or NaN
                const bool there = full(k) || s0 + k * GROUPS < n_split;
                m[k] = there ? m[k] : SQ_NEG_INF;
                n[k] = there ? n[k] : 0.0f;
#pragma unroll
                for (int d = 0; d < 4; ++d) v[k][d] = there ? v[k][d] : 0.0f;
            }
            fold(m, n, v);
        }
    };
    if constexpr (DEALT) {                                  // rounds as even as they go (uniform)
        const int per = (n_split + GROUPS - 1) / GROUPS, rounds = (per + AHEAD - 1) / AHEAD, ahead = (per + rounds - 1) / rounds;
        static_for<AHEAD + 1>([&](auto a) PF_INLINE {
            if constexpr (a > 0)
                if (ahead == a) take(a);
        });
    } else
        take(std::integral_constant<int, AHEAD>{});
    if constexpr (GROUPS > 1) {
        __shared__ __align__(16) float s_part[8][PART_STRIDE];
        if (lane == 0) {
            s_part[half][0] = M;
            s_part[half][1] = l;
        }
        *reinterpret_cast<f4 *>(&s_part[half][4 + 4 * lane]) = o;
        __syncthreads();
        if (group != 0) return;
        float m[GROUPS - 1], n[GROUPS - 1];
        f4 v[GROUPS - 1];
#pragma unroll
        for (int k = 0; k < GROUPS - 1; ++k) {              // (the row's other half waves)
            const float *p = s_part[half + 1 + k];
            m[k] = p[0];
            n[k] = p[1];
            v[k] = *reinterpret_cast<const f4 *>(p + 4 + 4 * lane);
        }
        fold(m, n, v);
    }
    if (row >= rows) return;
    const bool empty = !(l > 0.0f);
    const float inv = empty ? 0.0f : 1.0f / l;
    *reinterpret_cast<h4 *>(out + row * D + 4 * lane) = h4{(_Float16)(o[0] * inv), (_Float16)(o[1] * inv), (_Float16)(o[2] * inv),
                                                           (_Float16)(o[3] * inv)};
    if (lse && lane == 0) lse[row] = empty ? SQ_NEG_INF : M + logf(l);
}

// Waves per workgroup and the number of workgroups a unit's key blocks are dealt to.  A compute unit holds eight waves: one
// workgroup of eight (256 queries, half the staging per product) or two of four (128 queries, less padding of short or odd
// query blocks).  With u units and s shares the launch takes ceil(u s / slots) rounds of ceil(blocks / s) blocks each plus
// a fixed part (prologue, first loads, partial results: about six blocks' time), and the merge launch costs its own start
// and the partials' bytes.  In the shared-set form the number of kept keys is not known on the host: an eighth of the context
// is assumed (the rule only moves time, not results).  Eight waves unless four promise a tenth less.  Whole steps, us, the
// rule's shares / one share / half as many / twice as many, and all with eight / with four waves:
//   per query  32 heads x 1024 tokens x 32768 keys (8 waves, 2 shares)    608 /  950 / 948 / 652    605 / 623
//              32 heads x  150 tokens x 32768 keys (8, 8)                 184 /  902 / 275 / 205    184 / 186
//              2 x 12 heads x 333 tokens x 9001 keys (4, 7)              78.5 /  204 /  97 /  93     87 /  78
//              20 heads x   17 tokens x 22682 keys (4, 24)               68.5 /  413 /  69 /  77     79 /  69
//               5 heads x  600 tokens x 12000 keys (8, 17)               58.4 /  333 /  76 /  79     59 /  55
//   one set    32 heads x 1024 tokens x 32768 keys (8, 2)                 160 /  199 / 196 / 173    160 / 163
//              20 heads x  150 tokens x 20011 keys (8, 11)               42.1 /   83 /  44 /  51     42 /  43
//               8 heads x  512 tokens x 262144 keys, two-level (8, 16)    128 /  535 / 148 / 146    128 / 130
PfPlan prefill_plan(bool shared, const Shape &sh)
{
    const long long rows = (long long)sh.B * sh.H * sh.Lq;
    const long long fixed = ((long long)(shared ? (sh.L + 7) / 8 : sh.L) + PF_BN - 1) / PF_BN;
    const long long nblk = fixed + (sh.U + PF_BN - 1) / PF_BN;
    PfPlan best{8, 1};
    double best_cost = 0.0;
    for (int waves = 8; waves >= 4; waves -= 4) {
        const long long slots = 256 * 8 / waves, bm = pf_bm(waves);
        const long long units = (long long)sh.B * sh.H * ((sh.Lq + bm - 1) / bm);
        for (int s = 1; s == 1 || (s <= PF_MAX_SPLIT && s <= nblk && units * s <= 2 * slots); ++s) {
            const double rounds = (double)((units * s + slots - 1) / slots);
            const double cost = rounds * ((double)((nblk + s - 1) / s) + 6.0) + (s > 1 ? 3.0 + 1.5e-4 * (double)rows * s : 0.0);
            if (best_cost == 0.0 || cost < (waves < best.waves ? 0.9 * best_cost : best_cost)) {
                best = PfPlan{waves, s};
                best_cost = cost;
            }
        }
    }
    return best;
}

size_t prefill_partial_floats(bool shared, const Shape &sh)
{
    const int s = prefill_plan(shared, sh).n_split;
    if (shared && prefill_deal(sh, nullptr).units) return prefill_deal(sh, nullptr).words;
    return s > 1 ? (size_t)sh.B * sh.H * sh.Lq * s * PART_STRIDE : 0;
}

// Dealing costs a workgroup about a microsecond in front of its first load and the merge two, and pays where shares are long and heads
// keep different numbers of keys, which only the device knows.  Whole one-level steps, us, even / in proportion, by the share of the keys
// kept (heads alike up to 1/16, apart from 1/8 on):     1/32            1/16           0.09          1/8          0.2          0.3
//   20 heads x 257 tokens x  65536 keys            66.6 / 68.6    71.2 / 74.2    84.9 / 83.5   114 / 98    152 / 127    188 / 157
//   32       x 512        x 100000                  114 / 117      144 / 150      168 / 173    197 / 200   404 / 309    554 / 403
//   16       x 300        x 131072                 70.8 / 72.4    84.7 / 86.7     126 / 106    173 / 129   236 / 169    293 / 210
//   16       x 400        x 200000                 99.3 / 100.3    123 / 124      279 / 177    408 / 236   506 / 318    579 / 400
// Two-level steps, whose heads differ by a factor of three at the measured thresholds, us, even / in proportion, by heads x tokens x keys (blocks a share, an eighth
// of the context): 8 x 512 x 262144, 1/16 kept 104.7 / 98.8, 0.09 kept 123.7 / 114.5 (32); 4 x 300 x 200000 67.8 / 68.4 (12); 8 x 200 x
// 131072 69.0 / 67.6, 8 x 512 x 65536 73.5 / 74.0, one head x 512 x 262144 57.6 / 58.7 (8; one head's units keep the same keys).
PfDeal prefill_deal(const Shape &sh, float *ws)
{
    const PfPlan plan = prefill_plan(true, sh);
    const int bm = pf_bm(plan.waves);
    const long long units = (long long)sh.B * sh.H * ((sh.Lq + bm - 1) / bm);
    PfDeal d{};
    if (units > 64 || sh.B * sh.H == 1 || plan.n_split < PF_DEAL_MIN_SPLIT || (long long)sh.L < 8ll * PF_BN * PF_DEAL_MIN_BLOCKS * plan.n_split) return d;
    d.units = (int)units;
    d.shares = (int)units * plan.n_split;
    d.rows = std::min(bm, (sh.Lq + 7) / 8 * 8);
    const size_t floats = (size_t)d.shares * d.rows * PART_STRIDE;
    d.dealt = reinterpret_cast<int2 *>(ws + floats);
    d.words = floats + 2 * (size_t)units;
    return d;
}

namespace {

template <bool SHARED, int WAVES, int SELECT>
hipError_t launch_prefill_kernel(const void *q, const void *Kf, const void *Vf, const void *Ku, const void *Vu,
                                 const uint32_t *keep_mask, const uint32_t *table, const uint32_t *rows,
                                 const int32_t *blk_info, void *out, float *lse, float *partials, int n_split,
                                 const PfSelect &sel, const PfDeal &deal, const Shape &sh, hipStream_t s)
{
    constexpr int BM = pf_bm(WAVES);
    const int units = ((sh.Lq + BM - 1) / BM) * sh.H * sh.B * n_split;
    const dim3 grid((units + 7) / 8 * 8), block(64 * WAVES);
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (profile_pair(&ev0, &ev1))
        hipExtLaunchKernelGGL((prefill_attn_kernel<SHARED, WAVES, SELECT>), grid, block, 0, s, ev0, ev1, 0, (const _Float16 *)q,
                              (const _Float16 *)Kf, (const _Float16 *)Vf, (const _Float16 *)Ku, (const _Float16 *)Vu,
                              keep_mask, table, rows, blk_info, (_Float16 *)out, lse, partials, n_split, sh.B, sh.H, sh.L,
                              sh.C, sh.Lq, sh.U, sh.causal_user, sh.sm_scale, sel, deal);
    else
        hipLaunchKernelGGL((prefill_attn_kernel<SHARED, WAVES, SELECT>), grid, block, 0, s, (const _Float16 *)q,
                           (const _Float16 *)Kf, (const _Float16 *)Vf, (const _Float16 *)Ku, (const _Float16 *)Vu,
                           keep_mask, table, rows, blk_info, (_Float16 *)out, lse, partials, n_split, sh.B, sh.H, sh.L,
                           sh.C, sh.Lq, sh.U, sh.causal_user, sh.sm_scale, sel, deal);
    return hipGetLastError();
}

// The attention launch and, where the blocks are split, the merge launch.
template <bool SHARED, int SELECT>
hipError_t launch_prefill_kernels(const void *q, const void *Kf, const void *Vf, const void *Ku, const void *Vu,
                                  const uint32_t *keep_mask, const uint32_t *table, const uint32_t *rows,
                                  const int32_t *blk_info, void *out, float *lse, float *partials, const PfSelect &sel,
                                  const Shape &sh, hipStream_t s)
{
    const PfPlan plan = prefill_plan(SHARED, sh);
    const PfDeal deal = SHARED && !SELECT ? prefill_deal(sh, partials) : PfDeal{};
    const hipError_t e = plan.waves == 8 ? launch_prefill_kernel<SHARED, 8, SELECT>(q, Kf, Vf, Ku, Vu, keep_mask, table, rows, blk_info,
                                                                                    out, lse, partials, plan.n_split, sel, deal, sh, s)
                                         : launch_prefill_kernel<SHARED, 4, SELECT>(q, Kf, Vf, Ku, Vu, keep_mask, table, rows, blk_info,
                                                                                    out, lse, partials, plan.n_split, sel, deal, sh, s);
    if (e != hipSuccess || plan.n_split == 1) return e;
    const int bm = pf_bm(plan.waves);
    const size_t rows_out = (size_t)sh.B * sh.H * sh.Lq, n = deal.units ? (size_t)deal.units * deal.rows : rows_out;
    auto merge = [&](auto kernel, int groups) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n * groups + 7) / 8)), dim3(256), 0, s, partials, (_Float16 *)out, lse,
                           plan.n_split, n, PfMerge{deal, (sh.Lq + bm - 1) / bm, sh.B, sh.H, sh.Lq});
    };
    if (deal.units) {                                       // (a unit's shares are known there)
        rows_out >= 4096   ? merge(prefill_merge_kernel<8, 1, false, true>, 1)
        : rows_out >= 1024 ? merge(prefill_merge_kernel<8, 2, false, true>, 2)
                           : merge(prefill_merge_kernel<8, 8, false, true>, 8);
        return hipGetLastError();
    }
    // Several half waves per row where the rows are few; a half wave takes its shares in rounds of at most eight, as even as they go.
    // (3000 rows x 11 shares: two half waves 38.2 us a step, one 38.9; 1476 x 17: eight of them 6.3 us traced against 5.3 of a wave
    // per row.)
    const int groups = plan.n_split <= 8 || n >= 4096 ? 1 : plan.n_split <= 16 || n >= 1024 ? 2 : 8;
    const int each = (plan.n_split + groups - 1) / groups, rounds = (each + 7) / 8, ahead = (each + rounds - 1) / rounds;
    static_for<9>([&](auto a) {
        constexpr int A = a;
        if constexpr (A >= 2) {
            if (ahead != A) return;
            if (groups == 1 && rounds == 1) return merge(prefill_merge_kernel<A, 1, true, false>, 1);
            if constexpr (A >= 3)                           // (from 17 shares on)
                if (groups == 8) return merge(prefill_merge_kernel<A, 8, true, false>, 8);
            if constexpr (A >= 5) {                         // (from nine shares on: at least five in a round)
                if (groups == 1) return merge(prefill_merge_kernel<A, 1, false, false>, 1);
                return rounds == 1 ? merge(prefill_merge_kernel<A, 2, true, false>, 2) : merge(prefill_merge_kernel<A, 2, false, false>, 2);
            }
        }
    });
    return hipGetLastError();
}

}  // namespace

hipError_t launch_block_table(const BlockTable &bt, int H, hipStream_t s)
{
    hipLaunchKernelGGL(block_table_kernel, dim3(block_table_groups(bt.nblk), H), dim3(256), 0, s, bt);
    return hipGetLastError();
}

hipError_t launch_prefill_attn(const void *q, const void *Kf, const void *Vf, const void *Ku, const void *Vu,
                               const uint32_t *keep_mask, const BlockTable &bt, float *partials, void *out, float *lse,
                               const Shape &sh, hipStream_t s)
{
    return launch_prefill_kernels<false, 0>(q, Kf, Vf, Ku, Vu, keep_mask, bt.runs, bt.rows, bt.info, out, lse, partials, PfSelect{}, sh, s);
}

hipError_t launch_expand_ranges(DecodePlan plan, int32_t *idx, int rows, int L, hipStream_t s)
{
    // A wave's chain of records is what a launch over few rows waits for: 8 rows, 262144 keys and 16384 clusters, two launches,
    // 14.2 us with 16 workgroups per row, 9 with 64; from 32 rows on 16 fill the chip.
    const int slices = std::clamp(512 / rows, 16, 64);
    hipLaunchKernelGGL(expand_ranges_kernel, dim3(rows, slices), dim3(256), 0, s, plan, idx, L);
    return hipGetLastError();
}

hipError_t launch_prefill_attn_shared(const void *q, const void *Kf, const void *Vf, const void *Ku, const void *Vu,
                                      const int2 *hdr, const int32_t *key_idx, float *partials, void *out, float *lse,
                                      const Shape &sh, hipStream_t s)
{
    return launch_prefill_kernels<true, 0>(q, Kf, Vf, Ku, Vu, nullptr, reinterpret_cast<const uint32_t *>(key_idx), nullptr,
                                               reinterpret_cast<const int32_t *>(hdr), out, lse, partials, PfSelect{}, sh, s);
}

// Where the attention launch makes the kept set itself: where the records and the rows of a share's keys find room in LDS and the launch
// is about one round of workgroups, since a workgroup's few loads of scores (about 3 us, traced) cost less than a launch in front (5 to
// 7 us) and the two round trips to the list it leaves (2 us).  Whole steps, us, a launch of its own / here:
//   32 heads x 1024 tokens x 32768 keys, 1024 clusters 140.3 / 137.4    20 x 150 x 20011, 613 37.7 / 34.8    32 x 16 x 2000, 32 23.8 / 19.1
//    1 x 1024 x 32768, 1638  41.4 / 37.3     1 x 16 x 2000, 40  19.4 / 15.7     4 x 1024 x 8000, 400  43.4 / 39.5
//   2 x 32 x 500 x 20000, 500  127.9 / 124.9    32 x 16 x 32768, 1024  75.0 / 71.3    20 x 17 x 30000, 1500  49.8 / 47.9
// Every further round pays the 3 us again, and more where the scores come in many parts (the longer the prompt, the more, up to 512):
//    4 x 4096 x 8000, 400 (64 workgroups) 80.6 / 74.6    8 x 8192 x 8000, 400 (256) 294 / 289    one head x 16384 x 32768, 1024 (512 parts) 239 / 226
//   20 x 6000 x 4000, 200 (480, 25 parts) 98.9 / 98.2    12 x 10000 x 8000, 300 (480, 42) 150.9 / 151.0    3 x 32 x 1100 x 4000, 128 (480) 92.3 / 90.9
//    5 x 20000 x 16384, 1000 (395, 102) 229 / 239    3 x 40000 x 16384, 1000 (471, 157) 266 / 281    16 x 8192 x 16384, 1024 (512, 32) 262 / 268
//   20 x 8192 x 16384, 1024 (640) 338 / 349    32 x 8192 x 16384, 1024 (1024) 563 / 573    32 x 16384 x 16384, 1024 (2048) 989 / 1021
// Eight waves: 64 KB of rows beside 66 KB of tiles, one workgroup per compute unit as before; four: 12 KB, still two.
// A row's candidates: the same, up to 4096 clusters a head with eight waves (with four that many spill 61 registers) and not where the
// shares are dealt in proportion (their lengths come from the list in front).  Both-level steps, a launch of its own / here:
//   8 x 512 x 65536 3000  69.9 / 65.4    8 x 512 x 90000 4096  60.0 / 55.0    4 x 300 x 100000 4000  55.6 / 52.2    4 x 512 x 40000 1500  51.5 / 46.6
//   8 x 16 x 32768 2048  36.2 / 31.1    2 x 40 x 60000 2000  36.0 / 31.1    1 x 100 x 33000 700  35.2 / 30.8    1 x 3 x 130000 4096  40.5 / 37.8
//   24 x 4096 x 16384 1000 (384 workgroups) 201.5 / 197.9    32 x 4096 x 32768 2000 (512) 377.3 / 379.6    32 x 8192 x 16384 1000 (1024) 411 / 416
bool prefill_selects(const Shape &sh, bool candidates)
{
    const PfPlan plan = prefill_plan(true, sh);
    const long long blocks = ((long long)sh.L + PF_BN - 1) / PF_BN;
    if (candidates && prefill_deal(sh, nullptr).units) return false;
    if (sh.C > pf_select_max_c(plan.waves, candidates) || (blocks + plan.n_split - 1) / plan.n_split > pf_select_blocks(plan.waves)) return false;
    const long long bm = pf_bm(plan.waves), slots = 256 * 8 / plan.waves;
    const long long groups = (long long)sh.B * sh.H * ((sh.Lq + bm - 1) / bm) * plan.n_split;
    return groups <= slots || (8 * groups <= 15 * slots && (candidates || lookup_parts(sh.B * sh.H, sh.Lq, sh.C) <= 64));
}

hipError_t launch_prefill_attn_select(const void *q, const void *Kf, const void *Vf, const void *Ku, const void *Vu,
                                      const PfSelect &sel, float *partials, void *out, float *lse, const Shape &sh, hipStream_t s)
{
    if (!prefill_selects(sh, sel.cand_id != nullptr)) return hipErrorInvalidValue;
    auto launch = [&](auto selects) {
        return launch_prefill_kernels<true, selects>(q, Kf, Vf, Ku, Vu, nullptr, nullptr, nullptr, nullptr, out, lse, partials, sel, sh, s);
    };
    return sel.cand_id ? launch(std::integral_constant<int, 2>{}) : launch(std::integral_constant<int, 1>{});
}

}  // namespace sq
