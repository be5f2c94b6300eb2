// Shared device helpers for the gfx950 sparsified-FFN kernels (bf16 bit handling, 2:4 selection).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Tile rows per band of the workgroup -> tile map of the 256 x 256 tile kernels: the 32 workgroups that an XCD runs at a time
// cover GROUP tile rows x 32 / GROUP tile columns, and its L2 fetches the operand panels of exactly those rows and columns.
#ifndef SFFN_TILE_GROUP
#define SFFN_TILE_GROUP 4
#endif

namespace sffn {

__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }

// 16 bytes of a weight gradient, non-temporal: nothing reads it before the optimizer does, and stored the ordinary way the gradients push the operands that the other tiles share out of L2 and of
// the last-level cache.  Of the time with ordinary stores: 27 drawn steps 0.987, 14 on codes 0.978; with an update of the weights right behind the step 1.01 at 1 MB of gradient, 0.99 - 1.00 from 4 MB on.
// Activations (Y3, dX, y1, dy2, packed rows) the next kernel reads, and pays for it: vnm_spmm, then spmm24_fwd on its result, ordinary / non-temporal T = 256, D = 512, F = 1024 14.0 / 14.7 us,
// T = D = 1024, F = 4096 27.4 / 29.2, T = 8192, D = 2048, F = 8192 263 / 274; where they leave so all the same: stores_past(), results_past(), streams_between() in kernels.hpp.
typedef __attribute__((ext_vector_type(4))) uint32_t sffn_u32x4;
__device__ __forceinline__ void store_out(void* p, const uint4& w) { __builtin_nontemporal_store(__builtin_bit_cast(sffn_u32x4, w), reinterpret_cast<sffn_u32x4*>(p)); }
__device__ __forceinline__ void store_out(void* p, const float4& w) { store_out(p, __builtin_bit_cast(uint4, w)); }
// 16 bytes of an operand that is read once; PAST: non-temporal
template <bool PAST> __device__ __forceinline__ uint4 load_in(const void* p) {
    if (PAST) return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const sffn_u32x4*>(p)));
    return *reinterpret_cast<const uint4*>(p);
}
// What an epilogue leaves for the launches that follow, non-temporal where `stream` (the same in the whole launch: streams_between() in kernels.hpp): `stores` is called with the store to use.
// Without the barriers the compiler makes ordinary stores of both.
template <class F> __device__ __forceinline__ void store_between(bool stream, F stores) {
    if (stream) {
        asm volatile("" ::: "memory");
        stores([](auto* p, auto w) { if constexpr (sizeof(w) == 16) store_out(p, w); else __builtin_nontemporal_store(w, p); });
        asm volatile("" ::: "memory");
    } else {
        stores([](auto* p, auto w) { *reinterpret_cast<decltype(w)*>(p) = w; });
    }
}

// fp32 -> bf16 bits, round to nearest even, through gfx950's v_cvt_pk_bf16_f32 (checked against integer
// rounding on every bf16 pattern x tie / near-tie low halves, subnormals included; only NaN payloads differ).
typedef __attribute__((ext_vector_type(2))) float sffn_f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 sffn_bf16x2;
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {      // -> bf16(lo) | bf16(hi) << 16
    const sffn_f32x2 v = {lo, hi};
    const sffn_bf16x2 b = __builtin_convertvector(v, sffn_bf16x2);
    return __builtin_bit_cast(uint32_t, b);
}
__device__ __forceinline__ uint32_t f2bf(float f) { return f2bf2(f, 0.0f) & 0xFFFFu; }

// two real values -> two OCP E4M3 codes in the low 16 bits (first value in the low byte): one float32 product with inv = 1 / scale,
// saturation to +-448 (v_cvt_pk_fp8_f32 would give NaN above 464), one round-to-nearest-even
__device__ __forceinline__ uint32_t fp8_enc2(float a, float b, float inv) {
    const float ma = __builtin_fminf(__builtin_fmaxf(a * inv, -448.0f), 448.0f);
    const float mb = __builtin_fminf(__builtin_fmaxf(b * inv, -448.0f), 448.0f);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(ma, mb, 0, false) & 0xFFFFu;
}

// Largest magnitude seen by a wavefront -> *amax (device float32, atomic max on the bit pattern: non-negative floats order like their bits).
// m >= 0; every lane of the wavefront must call it.  At most one atomic per wavefront, and none when the value already there is
// at least as large (tens of thousands of wavefronts hitting one address serialise in L2: 1.5 ms instead of 0.03 for a pass over
// 128 MB; a stale read only costs a redundant atomic).
__device__ __forceinline__ void note_amax(float* amax, float m) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o, 64));
    if (amax && (threadIdx.x & 63) == 0) {
        unsigned int* p = reinterpret_cast<unsigned int*>(amax);
        if (__float_as_uint(m) > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, __float_as_uint(m));
    }
}

// The same for the epilogues of the fused fp8 step: 64 slots per tensor, 256 bytes apart (slot = workgroup id % 64), so that the reads and
// atomics of a launch spread over cache lines and L2 channels; the step's last launch folds them (amax_fold.hpp).
constexpr int kAmaxSlots = 64, kAmaxSlotStride = 64;      // floats

// 2:4 selection on one group of four bf16 (a0..a3 as 16-bit patterns): rank by magnitude
// descending, index ascending; the two first survive (Section 2.2 of the paper, with the tie rule
// of the packed-format contract).  Returns v0 | v1 << 16 (survivors in ascending position) and
// the metadata nibble p0 | p1 << 2.  SOFT: survivors move towards zero by the third-largest
// magnitude, evaluated in fp32 and rounded once to bf16.
// About 25 vector instructions (HARD) and 33 (SOFT) a group, where ranks out of six comparisons took 45 and 55: the four keys are distinct, so five of nine minima and maxima sort what is needed, and one byte
// permute fetches both survivors.  Eq. (1) of a small step, which prunes W1 itself: T = 512, D = 256, F = 1024 25.2 -> 24.5 us the step.
struct Selected24 { uint32_t v, nib, t; };       // survivors, positions, magnitude bits of the third
template <bool SOFT>
__device__ __forceinline__ Selected24 rank24(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
    // magnitude, then 3 - index: four keys in the order wanted
    const uint32_t k0 = ((a0 << 2) & 0x1FFFCu) | 3u, k1 = ((a1 << 2) & 0x1FFFCu) | 2u, k2 = ((a2 << 2) & 0x1FFFCu) | 1u, k3 = (a3 << 2) & 0x1FFFCu;
    auto lower = [](uint32_t p, uint32_t q) { return p < q ? p : q; };
    auto upper = [](uint32_t p, uint32_t q) { return p < q ? q : p; };
    const uint32_t high01 = upper(k0, k1), low01 = lower(k0, k1), high23 = upper(k2, k3), low23 = lower(k2, k3);
    const uint32_t x = lower(high01, high23), y = upper(low01, low23), first = upper(high01, high23), second = upper(x, y);
    const uint32_t i = first & 3u, j = second & 3u, both = upper(i, j) | (lower(i, j) << 16);     // 3 - p0, 3 - p1
    Selected24 r;
    r.v = __builtin_amdgcn_perm(a2 | (a3 << 16), a0 | (a1 << 16), 0x07060706u - (uint32_t)__mul24((int)both, 0x0202));
    r.nib = ((both | (both >> 14)) & 0xFu) ^ 0xFu;
    r.t = SOFT ? lower(x, y) >> 2 : 0u;
    return r;
}
template <bool SOFT>
__device__ __forceinline__ uint32_t select24(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t& nib) {
    const Selected24 s = rank24<SOFT>(a0, a1, a2, a3);
    nib = s.nib;
    if (!SOFT) return s.v;
    const float t = __uint_as_float(s.t << 16), f0 = __uint_as_float(s.v << 16), f1 = __uint_as_float(s.v & 0xFFFF0000u);
    return f2bf2(f0 - __builtin_copysignf(t, f0), f1 - __builtin_copysignf(t, f1));
}

// The survivors as float32 reals: bit copies widened (HARD) or a -/+ t evaluated in float32 (SOFT), not rounded to bf16.
template <bool SOFT>
__device__ __forceinline__ void select24_f32(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t& nib, float& f0, float& f1) {
    const Selected24 s = rank24<SOFT>(a0, a1, a2, a3);
    nib = s.nib;
    f0 = __uint_as_float(s.v << 16); f1 = __uint_as_float(s.v & 0xFFFF0000u);
    if (SOFT) {
        const float t = __uint_as_float(s.t << 16);
        f0 -= __builtin_copysignf(t, f0);
        f1 -= __builtin_copysignf(t, f1);
    }
}

// "Blocked" operand layout used between the kernels of the fused step: a K-contiguous matrix of
// 2-byte elements is cut into 1 KB blocks of 16 rows x 32 elements, block (r / 16, k / 32) stored at
// ((r / 16) * KC + k / 32) * 512 elements with KC = K / 32.  One wavefront-wide 16-byte-per-lane
// LDS-DMA load then moves exactly one contiguous block, which the L2 -> LDS path serves at close to
// twice the rate of eight separate 128-byte row segments.
__host__ __device__ __forceinline__ int64_t blk_off(int64_t r, int64_t k, int64_t KC) {
    return (((r >> 4) * KC + (k >> 5)) << 9) + ((r & 15) << 5) + (k & 31);
}
// fp8 operands use the same layout with a pair of 1-byte codes in the place of a 2-byte element (a block = 16 rows x 64 codes):
// blk_off(r, kbyte / 2, row bytes / 64) indexes 16-bit pairs.
// A transposed operand [rows, T] in the order in which v_mfma_f32_32x32x16_bf16 takes it (gemm_wgrad_wide_body.hpp): [T / 64][rows / 32][4 steps of 16 tokens]
// [64 lanes][8 tokens], lane = 32 (t / 8 % 2) + r % 32; element (r, t), t a multiple of 8.
__host__ __device__ __forceinline__ int64_t lane_off(int64_t r, int64_t t, int64_t R32) {
    return ((((t >> 6) * R32 + (r >> 5)) * 4 + ((t >> 4) & 3)) * 64 + ((t >> 3) & 1) * 32 + (r & 31)) * 8;
}

// The kept rows of a V:N:M activation (row = 4 block + position) in the same order, but the 32 rows of 8 blocks at the lanes kept_lane: any 8 lanes next to
// each other hold rows of 8 different blocks, which is what gemm_wgrad_wide_body.hpp's LDS accesses want.
__host__ __device__ __forceinline__ int kept_lane(int row) { return (row & 3) * 8 + (row >> 2); }
__host__ __device__ __forceinline__ int64_t kept_off(int64_t r, int64_t t, int64_t R32) { return lane_off((r & ~(int64_t)31) | kept_lane((int)(r & 31)), t, R32); }

// Metadata of a 2:4 matrix, blocked for the sparse matrix instruction: one 256-byte unit per (32 rows, 64 k).
// v_smfmac_f32_16x16x64_bf16 wants, in lane r % 16 + 16 q, the sixteen index bits of the row's survivors in k 16 q .. + 15; a unit stores, for each such
// lane, its two fragments of 16 rows as one 32-bit word (low half: the first) at byte 4 lane.  A wavefront therefore fetches a unit with one
// 4-byte-per-lane LDS-DMA load and reads it back with one conflict-free ds_read_b32.  mblk_off = byte address of the metadata byte covering k..k+7 of row r, KS = K / 64.
__host__ __device__ __forceinline__ int64_t mblk_off(int64_t r, int64_t k, int64_t KS) {
    return (((r >> 5) * KS + (k >> 6)) << 8) + (((k >> 4) & 3) << 6) + ((r & 15) << 2) + (((r >> 4) & 1) << 1) + ((k >> 3) & 1);
}

// The same for fp8 operands (v_smfmac_f32_16x16x128_fp8_fp8 wants a 32-bit index word per lane): one
// 512-byte unit per (32 rows, 128 k), row-major inside (16 bytes per row); a wavefront fetches its 32 rows of a stage with two
// contiguous 4-byte-per-lane loads.  m8blk_off = byte address of the metadata byte covering k..k+7 of row r, KS = K / 128.
__host__ __device__ __forceinline__ int64_t m8blk_off(int64_t r, int64_t k, int64_t KS) {
    return (((r >> 5) * KS + (k >> 7)) << 9) + ((r & 31) << 4) + ((k & 127) >> 3);
}

// Operands of the V:2:8 activation GEMM (gemm_vnm8.hip), written by the fused epilogues of eqs. (1), (4):
// survivors (element index of the pair of (token t, column block blk); F = d_ffn): 1 KB per (32 tokens, 64 hidden units)
__host__ __device__ __forceinline__ int64_t vcb_off(int64_t t, int64_t blk, int64_t F) {
    return ((((t >> 5) * (F >> 6) + (blk >> 3)) << 9) + ((t & 31) << 4) + ((blk & 7) << 1));
}
// metadata (byte address of the 4 bytes = 8 nibbles of (token t, 64 hidden units starting at column block blk8 * 8))
__host__ __device__ __forceinline__ int64_t mcb_off(int64_t t, int64_t blk8, int64_t F) {
    return (((t >> 6) * (F >> 6) + blk8) << 8) + ((t & 63) << 2);
}
// kept-column offsets, regrouped per (64 hidden units, token block) into the 8 words the transposing reads want (byte address of word 0)
__host__ __device__ __forceinline__ int64_t cixt_off(int64_t tb, int64_t blk8, int64_t n_tok_blocks) {
    return (blk8 * n_tok_blocks + tb) << 5;
}

// The same for the fp8 form of that kernel (a stage is 128 hidden units): byte address of the two codes of (token t, column block blk);
// of the 4 metadata bytes of (token t, 64 hidden units starting at column block blk8 * 8); of word 0 of the 16 offset words of
// (token block tb, 128 hidden units number s128)
__host__ __device__ __forceinline__ int64_t vcb8_off(int64_t t, int64_t blk, int64_t F) {
    return (((t >> 5) * (F >> 7) + (blk >> 4)) << 10) + ((t & 31) << 5) + ((blk & 15) << 1);
}
__host__ __device__ __forceinline__ int64_t mcb8_off(int64_t t, int64_t blk8, int64_t F) {
    return (((t >> 6) * (F >> 7) + (blk8 >> 1)) << 9) + ((t & 63) << 3) + ((blk8 & 1) << 2);
}
__host__ __device__ __forceinline__ int64_t cixt8_off(int64_t tb, int64_t s128, int64_t n_tok_blocks) {
    return (s128 * n_tok_blocks + tb) << 6;
}

// In two steps, since the epilogue's stores would otherwise stand between the early-out read and its use (loads and stores share one in-order
// counter): amax_slot_peek reads the workgroup's slot before the stores are issued, note_amax_slots_seen compares against that value.
__device__ __forceinline__ uint32_t amax_slot_peek(const float* slots) {
    if (!slots) return 0u;
    const unsigned int* p = reinterpret_cast<const unsigned int*>(slots + (((blockIdx.y * gridDim.x + blockIdx.x) & (kAmaxSlots - 1)) * kAmaxSlotStride));
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void note_amax_slots_seen(float* slots, float m, uint32_t seen) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o, 64));
    if (slots && (threadIdx.x & 63) == 0 && __float_as_uint(m) > seen)
        atomicMax(reinterpret_cast<unsigned int*>(slots + (((blockIdx.y * gridDim.x + blockIdx.x) & (kAmaxSlots - 1)) * kAmaxSlotStride)), __float_as_uint(m));
}

// Two survivors per 8 columns leave at most two per aligned group of four, so a V:2:8 row block is
// also two plain 2:4 groups.  Inputs: v = the two survivors (low half first), nib = their positions
// among the four kept columns, cw = the four kept column offsets (one per byte).  Outputs: the two
// packed groups (empty slots are +0 at unused positions) and their metadata byte.
__device__ __forceinline__ void vnm_block_to_24(uint32_t v, uint32_t nib, uint32_t cw, uint32_t& a, uint32_t& b, uint32_t& mbyte) {
    const uint32_t o0 = (cw >> (8 * (nib & 3u))) & 0xFFu, o1 = (cw >> (8 * (nib >> 2))) & 0xFFu;   // o0 < o1
    const uint32_t v0 = v & 0xFFFFu, v1 = v >> 16;
    const bool lo0 = o0 < 4, lo1 = o1 < 4;            // survivor in columns 0-3?  (lo1 implies lo0)
    // low group: both survivors | only the first (kept next to an empty slot at position 3, or after one at 0) | none
    const uint32_t a_split = (o0 < 3) ? v0 : (v0 << 16), na_split = (o0 < 3) ? (o0 | (3u << 2)) : (3u << 2);
    a = lo1 ? v : (lo0 ? a_split : 0u);
    const uint32_t na = lo1 ? (o0 | (o1 << 2)) : (lo0 ? na_split : 0x4u);
    // high group: both | only the second | none
    const uint32_t q = o1 - 4;
    const uint32_t b_split = (q > 0) ? (v1 << 16) : v1, nb_split = (q > 0) ? (q << 2) : 0x4u;
    b = !lo0 ? v : (!lo1 ? b_split : 0u);
    const uint32_t nb = !lo0 ? ((o0 - 4) | (q << 2)) : (!lo1 ? nb_split : 0x4u);
    mbyte = na | (nb << 4);
}

// lane i <- lane i + N inside a row of 16 lanes (0 past the row's end): one DPP move instead of an LDS permute
template <int N>
__device__ __forceinline__ uint32_t row_shl(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x100 | N, 0xF, 0xF, true);
}

// the same with any control word: permutations inside groups of 4, mirrored groups of 8, rotation of a row of 16 (| 1 .. 15, lane i <- lane i - n)
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kQuadXor3 = 0x1B, kRowHalfMirror = 0x141, kRowRor = 0x120;
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// bitwise OR over every aligned group of 8 lanes, in all of them
__device__ __forceinline__ uint32_t or_of_8(uint32_t x) {
    x |= dpp<kQuadXor1>(x);
    x |= dpp<kQuadXor2>(x);
    return x | dpp<kRowHalfMirror>(x);
}

// lane I of every aligned group of 8 lanes, in all of them
template <int I>
__device__ __forceinline__ uint32_t bcast_of_8(uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (I << 5) | 0x18); }

// y1 at y2's kept slots, as the fused epilogues write and read it: 2 KB runs of (64 tokens x 8 column blocks);
// index in 32-bit words of (token t, column block blk), F = d_ffn.
__host__ __device__ __forceinline__ int64_t ykept_off(int64_t t, int64_t blk, int64_t F) {
    return ((((t >> 6) * (F >> 6) + (blk >> 3)) << 6) + (t & 63)) * 8 + (blk & 7);
}

}  // namespace sffn
