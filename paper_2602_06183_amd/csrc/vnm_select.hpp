// eq. (2) and the two choices of the V:N:M rule (Section 2.3) on values in registers: used by the epilogues of eqs. (1), (4) (gemm_v2_body.hpp) and by the
// stand-alone compressor (vnm_general.hip).
#pragma once
#include "common.hpp"

namespace sffn {

// max(x, 0) in one instruction, 0 for NaN.  (As a comparison, as fmaxf or with an infinity that the compiler sees: two, the first to quiet a NaN.)
__device__ __forceinline__ float relu1(float x) {
    float inf = __builtin_inff();
    asm("" : "+s"(inf));
    return __builtin_amdgcn_fmed3f(x, 0.0f, inf);
}
// eq. (2): bf16 bits -> max(y, 0)^2 rounded to bf16 (RNE), one value or the two of a word
__device__ __forceinline__ uint32_t sqrelu16(uint32_t y) {
    const float r = relu1(bf2f(y));
    return f2bf(r * r);
}
__device__ __forceinline__ uint32_t sqrelu2(uint32_t w) {
    const float a = relu1(__uint_as_float(w << 16)), b = relu1(__uint_as_float(w & 0xFFFF0000u));
    return f2bf2(a * a, b * b);
}
// The 2:4 choice of the V:N:M epilogues among the four kept columns of a block, for values that are not negative (y2): the two largest, ties to the lower
// column, in ascending column order as low | high << 16.  A key is the value in its upper half over tag[i], which falls with i, so that the order of the
// keys is the order of the rule; keys come back with the values.  (With ranks out of six comparisons: 50 instructions instead of 20.)
__device__ __forceinline__ uint32_t pick24_pos(uint32_t y01, uint32_t y23, const uint32_t (&tag)[4], uint32_t& low, uint32_t& high) {
    const uint32_t k0 = (y01 << 16) | tag[0], k1 = (y01 & 0xFFFF0000u) | tag[1], k2 = (y23 << 16) | tag[2], k3 = (y23 & 0xFFFF0000u) | tag[3];
    const uint32_t a = k0 > k1 ? k0 : k1, b = k0 > k1 ? k1 : k0, c = k2 > k3 ? k2 : k3, d = k2 > k3 ? k3 : k2;
    const uint32_t first = a > c ? a : c, ac = a > c ? c : a, bd = b > d ? b : d, second = ac > bd ? ac : bd;
    const bool ordered = (uint16_t)first > (uint16_t)second;      // the larger tag is the lower column
    low = ordered ? first : second;
    high = ordered ? second : first;
    return __builtin_amdgcn_perm(high, low, 0x07060302u);         // upper halves
}
// Is the score of this lane's column among the four largest of its block of M lanes (ties to the lower column)?  sc: float32 bits, not negative.
__device__ __forceinline__ bool keep4_of_8(uint32_t sc, int lane) {
    const uint32_t a1 = lane & 1, a2 = (lane >> 1) & 1, a4 = (lane >> 2) & 1;         // lane ^ k is a lower column if the top bit of k is set in lane
    const uint32_t m7 = dpp<kRowHalfMirror>(sc);
    return (dpp<kQuadXor1>(sc) + a1 > sc) + (dpp<kQuadXor2>(sc) + a2 > sc) + (dpp<kQuadXor3>(sc) + a2 > sc) + (m7 + a4 > sc) + (dpp<kQuadXor1>(m7) + a4 > sc) +
               (dpp<kQuadXor2>(m7) + a4 > sc) + (dpp<kQuadXor3>(m7) + a4 > sc) < 4;
}
// (M >= 16: the largest of the block four times over; M - 1 comparisons are more)
template <int M>
__device__ __forceinline__ bool keep4_of(uint32_t sc, int lane) {
    const int c = lane & (M - 1);
    int mine = (int)sc;
    bool kept = false;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        int x = mine, o;
        o = (int)dpp<kRowRor | 8>((uint32_t)x); x = x > o ? x : o;
        o = (int)dpp<kRowRor | 4>((uint32_t)x); x = x > o ? x : o;
        o = (int)dpp<kRowRor | 2>((uint32_t)x); x = x > o ? x : o;
        o = (int)dpp<kRowRor | 1>((uint32_t)x); x = x > o ? x : o;
        if (M >= 32) { o = __builtin_amdgcn_ds_swizzle(x, (0x10 << 10) | 0x1F); x = x > o ? x : o; }
        if (M == 64) { o = __shfl_xor(x, 32, 64); x = x > o ? x : o; }
        const unsigned long long eq = __ballot(mine == x);
        const uint32_t half = (uint32_t)(lane < 32 ? eq : eq >> 32);
        const int first = M == 64 ? __builtin_ctzll(eq) : M == 32 ? __builtin_ctz(half) : __builtin_ctz((half >> (lane & 16)) & 0xFFFFu);
        const bool me = first == c;
        kept |= me;
        mine = me ? -1 : mine;
    }
    return kept;
}

}  // namespace sffn
