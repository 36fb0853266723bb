// Shared by the prefill lookup kernels.
#pragma once
#include "sq_common.hpp"

namespace sq {

// Rows of 256 B staged unpadded by the load-to-LDS instruction (a wave writes four whole rows); 16-byte chunk c of row r sits
// at slot c ^ (r % 16), applied on the global side, so the operand reads (32 rows at one chunk index) are free of conflicts.
typedef __attribute__((address_space(3))) void *lk_lptr_t;
__device__ __forceinline__ void lk_stage(const char *base, uint32_t off, uint32_t lds)   // base, lds: uniform
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0");
}

constexpr int LK_MC = 128;                   // clusters per workgroup of the averaging kernel (four waves x 32)
constexpr int LK_MT = 64;                    // tokens per staged tile
constexpr int LK_MEAN_GROUPS = 512;          // workgroups of it that there should be: two per compute unit

// Parts the tokens of a row with C clusters are dealt to where (sequence, head) x blocks of clusters alone are few; and, for
// candidates, whose number n the device alone knows, the length of a row's partial sums, [parts of n][n] in front: room for n = C_all
// in one part and for any n whose parts are more (parts * blocks * BH <= LK_MEAN_GROUPS).
__host__ __device__ inline int lookup_mean_parts(int BH, int Lq, int C)
{
    const int blocks = (C + LK_MC - 1) / LK_MC, tiles = (Lq + LK_MT - 1) / LK_MT, groups = LK_MEAN_GROUPS / BH;
    const int p = blocks > 0 ? groups / blocks : 1;
    return p < 1 ? 1 : p < tiles ? p : tiles;
}
__host__ __device__ inline size_t lookup_cand_stride(int BH, int C_all) { return (size_t)C_all + LK_MEAN_GROUPS * LK_MC / BH; }

// The least raw score x that passes exp2((x - m) c2) > thr, the test of Eq. 1's scores against T * D with m the row's largest
// score: exactly the boundary of that float expression, so that a score which equals the threshold is dropped.  (thr < 0:
// everything; thr >= 1 or not a number: nothing -- NaN, which no comparison passes.)  The differences that pass are an interval
// [d, 0]; d is bisected from a bracket around the logarithm, wide enough for the rounding of the exponential (relative to d that
// grows as 1 / |d c2|), or from all floats where the bracket does not hold it.  7 to 10 steps, once per token and workgroup.
__device__ __forceinline__ float lk_least_kept(float m, float thr, float c2)
{
    if (thr < 0.0f) return SQ_NEG_INF;
    if (!(thr < 1.0f)) return __builtin_nanf("");
    auto passes = [&](uint32_t u) { return __builtin_amdgcn_exp2f(-__builtin_bit_cast(float, u) * c2) > thr; };
    const float l = thr > 0.0f ? fmaxf(-log2f(thr), 0x1p-26f) : 126.0f;   // (positive, also for the float below 1)
    const uint32_t at = __builtin_bit_cast(uint32_t, fminf(l / c2, 3e38f)), w = (uint32_t)fminf(16.0f + 16.0f / l, 4e6f);
    uint32_t lo = at > w ? at - w : 0u, hi = min(at + w, 0x7f800000u);   // (bit patterns of -d; -0 passes, -inf does not)
    if (!passes(lo)) lo = 0u;
    if (passes(hi)) hi = 0x7f800000u;
    while (hi - lo > 1u) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (passes(mid)) lo = mid;
        else hi = mid;
    }
    // x passes iff fl(x - m) >= d: the least one lies next to m + (d + the float below it) / 2
    const float d = -__builtin_bit_cast(float, lo);
    const double at_x = (double)m + 0.5 * ((double)d - (double)__builtin_bit_cast(float, hi));
    float x = nextafterf((float)at_x, SQ_NEG_INF);
    for (int i = 0; i < 2; ++i)
        if (!(x - m >= d)) x = nextafterf(x, __builtin_inff());
    return x;
}

}  // namespace sq
