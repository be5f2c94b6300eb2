// A contraction shared by several workgroups of one output tile (eqs. (3), (7) on few tokens: 64 x 64 tiles of a T = 64 call occupy N / 64 of the 256
// CUs, and what bounds them is the rate at which one CU can be fed).  Split s contracts its own range of stages; every workgroup leaves its float32
// sums in memory and counts itself in; those that find the others there add all of them in the order of the splits, so the result does not depend
// on who was last, and go on to the output.  Nothing waits.  The counters are zero before the launch (the step's preparing launch clears them)
// and zero after it.
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "lds_dma.hpp"

namespace sffn {

// The sums travel as agent-scope atomics (written through to memory and read from there: every XCD has its own L2), which the count follows once they are
// complete.  A fence would write back and invalidate the whole L2 instead, for every wavefront: 250 us for a contraction of 130.

// Sum over the four wavefronts of a workgroup, which share a 64 x 64 tile (64 sums a lane, in `acc`), in ascending order.  Wavefront w is left with its quarter of the
// tile's sums, q[16] (accumulators 16 w .. 16 w + 15 of a lane in the order [a][b][r]).  smem: kJoin4 bytes, which other wavefronts may still be reading afterwards.
constexpr int kJoin4 = 4 * 16 * 1024;
__device__ __forceinline__ void join4(const f32x16 (&acc)[2][2], unsigned char* smem, int wave, int lane, float (&q)[16]) {
    f32x4* const part = reinterpret_cast<f32x4*>(smem) + lane;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const f32x16& v = acc[k >> 3][k >> 2 & 1];
        const int r = (k & 3) * 4;
        part[(wave * 16 + k) * 64] = f32x4{v[r], v[r + 1], v[r + 2], v[r + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f32x4 sum = part[(wave * 4 + k) * 64];
#pragma unroll
        for (int g = 1; g < 4; ++g) sum += part[(g * 16 + wave * 4 + k) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) q[4 * k + r] = sum[r];
    }
}

// The same over the workgroups that share the tile too.  false: the others are not there yet, the wavefront is done.  Every wavefront counts in by itself when its quarter is out and sums that
// quarter if it is the last to come.  The counts bound it: an atomic takes its line for 6 ns, and 32 tiles of 8 splits that count on one line are 1.5 us.  Forward calls of T = 64, D = 2048,
// F = 8192 (32 tiles, 8 splits) and T = 128 (64, 4): one count a workgroup, on consecutive words 21.1 and 23.2 us; on a line a tile 20.3, 22.9; one a wavefront on those lines 19.8, 22.6,
// on consecutive words 25.1, 27.0.  Eight splits' loads at a time instead of four: 0.4 us of the first.
__device__ __forceinline__ bool split_join4(const f32x16 (&acc)[2][2], unsigned char* smem, const Split& sp, int tile, int s, int wave, int lane, float (&q)[16]) {
    join4(acc, smem, wave, lane, q);
    unsigned long long* const p = reinterpret_cast<unsigned long long*>(sp.part) + ((int64_t)tile * sp.n * 4 + wave) * (8 * 64) + lane;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        __hip_atomic_store(p + (s * 4 * 8 + k) * 64, (unsigned long long)__float_as_uint(q[2 * k]) | ((unsigned long long)__float_as_uint(q[2 * k + 1]) << 32), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // a byte of the tile's word for each quarter; consecutive tiles on different lines
    unsigned* const count = sp.count + (tile & 31) * 32 + (tile >> 5);
    const unsigned one = 1u << (8 * wave);
    unsigned before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(count, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uniform((int)before) >> (8 * wave) & 0xFF) + 1 != sp.n) return false;
    asm volatile("" ::: "memory");       // relaxed loads of other addresses: nothing else keeps the compiler from reading the sums before the count
    if (lane == 0) __hip_atomic_fetch_sub(count, one * (unsigned)sp.n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int k = 0; k < 16; ++k) q[k] = 0.0f;
    auto add = [&](int g0, auto batch) {                    // the loads of `batch` splits at a time
        constexpr int B = decltype(batch)::value;
        unsigned long long v[B][8];
#pragma unroll
        for (int g = 0; g < B; ++g)
#pragma unroll
            for (int k = 0; k < 8; ++k)
                v[g][k] = g0 + g < sp.n ? __hip_atomic_load(p + ((g0 + g) * 4 * 8 + k) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
#pragma unroll
        for (int g = 0; g < B; ++g)
#pragma unroll
            for (int k = 0; k < 8; ++k) { q[2 * k] += __uint_as_float((uint32_t)v[g][k]); q[2 * k + 1] += __uint_as_float((uint32_t)(v[g][k] >> 32)); }
    };
    if (sp.n <= 4) add(0, std::integral_constant<int, 4>());
    else for (int g0 = 0; g0 < sp.n; g0 += 8) add(g0, std::integral_constant<int, 8>());
    return true;
}

// The quarter's output: accumulators 16 w .. of the layout [a][b][r] are the 32 x 32 sub-tile (a, b) = (w / 2, w % 2); rows of 64 bytes through LDS
__device__ __forceinline__ void store_quarter(const float (&q)[16], float alpha, unsigned char* smem, int wave, int lane, uint16_t* __restrict__ out, int64_t ldo, int i0, int j0,
                                              int Ra, int N) {
    constexpr int EP = 32 * 2 + 16;
    const int l32 = lane & 31, lh = lane >> 5;
    unsigned char* const scratch = smem + wave * (32 * EP);
#pragma unroll
    for (int r = 0; r < 16; ++r) *reinterpret_cast<uint16_t*>(scratch + (8 * (r >> 2) + 4 * lh + (r & 3)) * EP + l32 * 2) = (uint16_t)f2bf(q[r] * alpha);
    wave_lds_sync();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int e = lane + 64 * p, row = e >> 2, ch = e & 3;
        const int i = i0 + (wave >> 1) * 32 + row, j = j0 + (wave & 1) * 32 + ch * 8;
        if (i < Ra && j < N) *reinterpret_cast<uint4*>(out + (int64_t)i * ldo + j) = *reinterpret_cast<const uint4*>(scratch + row * EP + ch * 16);
    }
}

}  // namespace sffn
