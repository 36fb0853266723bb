// Kept clusters -> rows of the key-index list (Section 4.2), written by a whole workgroup.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sq {

// Key-index entries of the kept clusters rec[0..n) = (first key, keys, position in the row's list) of a slice: eight
// lanes per cluster, so 8 x (waves of the workgroup) clusters are written per round.  (A wave per cluster took eight
// rounds for a 128-cluster slice of a row that keeps everything, and the launch waited 1.6 us for that row's workgroups;
// measured on the whole step at 32 heads x 32K keys: a wave per cluster 28.10 us, 16 lanes 27.82, 8 lanes 27.70, the
// group width chosen by the number of clusters 27.81.)  The eight lanes write the first 64 keys of their cluster; the
// rest of a longer cluster is written by the whole wave.  Called by every thread of the workgroup.
constexpr int KI_WRITE_SH = 3;                                       // log2 of the lanes per cluster
__device__ __forceinline__ void write_key_index(const int4 *rec, int n, int32_t *__restrict__ idx_row, int L, int threads)
{
    constexpr int LPC = 1 << KI_WRITE_SH, PER_WAVE = 64 / LPC;
    const int lane = threadIdx.x & 63;
    for (int c0 = (threadIdx.x >> 6) * PER_WAVE; c0 < n; c0 += (threads >> 6) * PER_WAVE) {   // (wave-uniform bounds)
        const int c = c0 + (lane >> KI_WRITE_SH);
        const int4 rc = c < n ? rec[c] : make_int4(0, 0, 0, 0);
        const int head = min(rc.y, 64);
        for (int j = lane & (LPC - 1); j < head && rc.z + j < L; j += LPC)
            idx_row[rc.z + j] = max(0, min(rc.x + j, L - 1));        // malformed offsets stay in the tensor
        unsigned long long big = __ballot(rc.y > 64);
        while (big) {                                                // wave-uniform; rare
            const int src = __builtin_ctzll(big);                    // a lane of the long cluster's group
            big &= ~(((1ull << LPC) - 1ull) << (src & ~(LPC - 1)));
            const int bx = __shfl(rc.x, src), by = __shfl(rc.y, src), bz = __shfl(rc.z, src);
            for (int j = 64 + lane; j < by && bz + j < L; j += 64) idx_row[bz + j] = max(0, min(bx + j, L - 1));
        }
    }
}

}  // namespace sq
