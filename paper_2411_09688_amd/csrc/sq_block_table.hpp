// The block table of the masked prefill attention: per (head, 64-key block) the runs of keys that share a cluster (clusters
// are contiguous key ranges, so a block is a few runs: three at 32 keys per cluster).
//   runs[h, blk, i]   cluster | first key of the run in the block << 16 | (keys - 1) << 22, ascending
//   rows[h, blk]      the same for up to PF_ROW_RUNS runs in the form the attention kernel uses, groups of four runs, PF_ROW_GROUP
//                     words each: [0..3] cluster relative to the block's first (31, a window bit that is never set, for none),
//                     [4..7] / [8..11] the run's keys for lanes 0..31: bit 8 a + i = key 32 t + 8 a + i, t = 0 / 1,
//                     [12..15] / [16..19] for lanes 32..63: key 32 t + 8 a + 4 + i (i < 4: see the accumulator layout there)
//   info[h, blk]      first cluster | min(span of cluster ids, 30) << 16 | n runs << 21 | wide << 31; wide: the span does
//                     not fit the 31-bit window of mask bits (a block that crosses many empty clusters)
// Keys that no cluster covers (before offsets[0] or from offsets[C] on) belong to no run.  One wave per block: a 64-way
// search for the first key's cluster, then the keys are placed among the next 64 cluster starts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sq {

constexpr int PF_BN = 64;                 // keys per block
constexpr int PF_ROW_RUNS = 12, PF_ROW_GROUP = 20, PF_ROW_WORDS = 64;
struct BlockTable {
    const int32_t *offsets;               // [H, C + 1]
    uint32_t *runs, *rows;                // [H, nblk, PF_BN], [H, nblk, PF_ROW_WORDS]
    int32_t *info;                        // [H, nblk]
    int C, L, nblk;
};

// It depends on the offsets alone, so a whole step makes it in extra workgroups of the lookup's first launch.  That lengthens
// that launch by about what a launch of its own takes (12 us at 32 heads x 512 blocks), but saves the launch: whole steps, with a
// launch of its own / in the lookup's, us: 2 x 12 heads x 333 tokens x 9001 keys 80.2 / 77.2, 8 heads x 60 tokens x 32K keys
// 56.7 / 53.6, 16 heads x 28 tokens x 2400 keys 31.6 / 25.5, 32 heads x 1024 tokens x 32K keys the same (603 / 604).
// A workgroup makes the entries of PF_TAB_BLOCKS blocks, whatever its number of waves.
constexpr int PF_TAB_BLOCKS = 16;
__host__ __device__ inline int block_table_groups(int nblk) { return (nblk + PF_TAB_BLOCKS - 1) / PF_TAB_BLOCKS; }

__device__ __forceinline__ void block_table_entry(const BlockTable &bt, int h, int blk, int lane)
{
    const int C = bt.C, L = bt.L, nblk = bt.nblk;
    const int32_t *off = bt.offsets + (size_t)h * (C + 1);
    const int j0 = blk * PF_BN, j = j0 + lane;
    int lo = -1, hi = C + 1;                             // the last c with off[c] <= j0 (-1: none) lies in [lo, hi)
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) >> 6, at = lo + (lane + 1) * step;
        const bool le = at < hi && off[min(at, C)] <= j0;
        lo += __popcll(__ballot(le)) * step;
        hi = min(hi, lo + step);
    }
    const int nx = lo + 1 + lane;
    const int start = nx <= C ? off[nx] : 0x7fffffff;    // starts of the 64 clusters after it
    int pos = 0;                                         // how many of them are at or before this lane's key
#pragma unroll
    for (int step = 32; step > 0; step >>= 1)
        if (__shfl(start, pos + step - 1) <= j) pos += step;
    if (__shfl(start, pos) <= j) ++pos;
    int c = lo + pos;
    if (__ballot(pos == 64) != 0ull) {                   // more than 64 cluster starts in the block: search for each key
        int a = lo, b = C + 1;
        while (b - a > 1) {
            const int mid = (a + b) >> 1;
            if (off[mid] <= j) a = mid;
            else b = mid;
        }
        c = a;
    }
    const bool covered = c >= 0 && c < C && j < L;
    if (!covered) c = 0x7fffffff;
    const int before = __shfl_up(c, 1);
    const bool change = lane == 0 || c != before;
    const unsigned long long cuts = __ballot(change), heads = __ballot(change && covered);
    const int n = __popcll(heads);
    const unsigned long long later = lane == 63 ? 0ull : cuts >> (lane + 1);
    const int len = later ? __ffsll((long long)later) : 64 - lane;   // keys up to the next cut
    uint32_t *dst = bt.runs + ((size_t)h * nblk + blk) * PF_BN;
    const unsigned long long in = __ballot(covered);
    const int first = n ? __shfl(c, __ffsll((long long)heads) - 1) : 0;
    const int last = n ? __shfl(c, 63 - __clzll((long long)in)) : 0;
    uint32_t *row = bt.rows + ((size_t)h * nblk + blk) * PF_ROW_WORDS;
    auto put = [&](int slot, uint32_t rel, unsigned long long keys) {
        uint32_t *g = row + (slot >> 2) * PF_ROW_GROUP + (slot & 3);
        g[0] = rel;
        g[4] = (uint32_t)keys & 0x0f0f0f0fu;
        g[8] = (uint32_t)(keys >> 32) & 0x0f0f0f0fu;
        g[12] = (uint32_t)(keys >> 4) & 0x0f0f0f0fu;
        g[16] = (uint32_t)(keys >> 36) & 0x0f0f0f0fu;
    };
    if (change && covered) {
        const int slot = __popcll(heads & ((1ull << lane) - 1ull));
        dst[slot] = (uint32_t)c | (uint32_t)lane << 16 | (uint32_t)(len - 1) << 22;
        if (slot < PF_ROW_RUNS) put(slot, (uint32_t)min(c - first, 31), (~0ull >> (64 - len)) << lane);
    }
    if (lane >= n && lane < PF_ROW_RUNS) put(lane, 31u, 0ull);
    if (lane == 0) {
        const int span = max(last - first, 0);
        bt.info[(size_t)h * nblk + blk] = first | (min(span, 30) << 16) | (n << 21) | (span >= 31 ? (int)0x80000000 : 0);
    }
}

__device__ __forceinline__ void block_table_part(const BlockTable &bt, int h, int group, int waves)
{
    const int lane = threadIdx.x & 63;
    for (int i = threadIdx.x >> 6; i < PF_TAB_BLOCKS; i += waves) {
        const int blk = group * PF_TAB_BLOCKS + i;
        if (blk < bt.nblk) block_table_entry(bt, h, blk, lane);
    }
}

}  // namespace sq
