// Bodies of the scans that prepare the operands of the contractions: used by their own kernels (prune24.hip, vnm.hip) and, several in one
// launch, by the step's prologue (prologue.hip).  bx, by, bz: the workgroup's place in the scan's own grid; smem: LDS of the stated size.
#pragma once
#include "common.hpp"

namespace sffn {

constexpr int kTransposeLds = 64 * (64 + 2) * 2, kPruneColsLds = 128 * (64 + 2) * 2;

// out[c, r] = in[r, c]; R, C multiples of 64.
// blocked = 2: out in the order of lane_off (common.hpp), out_same as for 1.
// blocked = 1: out (the transpose) and, when given, out_same (a copy of `in`) are written in the blocked
// operand layout instead of row-major.
// in_perm: row r of the matrix is row in_perm[r] of `in`; negative: a zero row.
__device__ __forceinline__ void transpose_bf16_body(void* smem, int bx, int by, const uint16_t* __restrict__ in, int64_t R, int64_t C, int64_t ld,
                                                    uint16_t* __restrict__ out, int blocked, uint16_t* __restrict__ out_same, const int32_t* __restrict__ in_perm) {
    uint16_t (*tile)[64 + 2] = reinterpret_cast<uint16_t (*)[64 + 2]>(smem);
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)by * 64, c0 = (int64_t)bx * 64;
    uint4 w[2];                              // both loads before either is waited for, so no branch around them
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 256 * i, rr = e >> 3, seg = e & 7;
        int64_t rs = r0 + rr;
        if (in_perm) rs = in_perm[rs];
        w[i] = *reinterpret_cast<const uint4*>(in + (rs < 0 ? 0 : rs) * ld + c0 + seg * 8);
        if (rs < 0) w[i] = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 256 * i, rr = e >> 3, seg = e & 7;
        uint32_t* p = reinterpret_cast<uint32_t*>(&tile[rr][seg * 8]);
        p[0] = w[i].x; p[1] = w[i].y; p[2] = w[i].z; p[3] = w[i].w;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 256 * i;
        int cc, rs;                          // output row (a column of `in`) and first of 8 source rows
        if (blocked == 2) { cc = ((e >> 8) & 1) * 32 + (e & 31); rs = ((e >> 6) & 3) * 16 + ((e >> 5) & 1) * 8; }
        else if (blocked) { const int bk = e >> 6, l = e & 63; cc = (bk >> 1) * 16 + (l >> 2); rs = (bk & 1) * 32 + (l & 3) * 8; }
        else { cc = e >> 3; rs = (e & 7) * 8; }
        if (out) {                           // (out = nullptr: only the blocked copy of `in` is wanted)
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = tile[rs + 2 * j][cc] | ((uint32_t)tile[rs + 2 * j + 1][cc] << 16);
            uint16_t* dst = blocked == 2 ? out + lane_off(c0 + cc, r0 + rs, C / 32) : blocked ? out + blk_off(c0 + cc, r0 + rs, R / 32) : out + (c0 + cc) * R + r0 + rs;
            *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
        }
        if (out_same) {
            const int bk = e >> 6, l = e & 63, rr = (bk >> 1) * 16 + (l >> 2), cs = (bk & 1) * 32 + (l & 3) * 8;
            const uint32_t* p = reinterpret_cast<const uint32_t*>(&tile[rr][cs]);
            *reinterpret_cast<uint4*>(out_same + blk_off(r0 + rr, c0 + cs, C / 32)) = make_uint4(p[0], p[1], p[2], p[3]);
        }
    }
}

// ---- groups run along the strided axis: S[r,k] = src[k*ld + r] ---------------------------------
// A workgroup takes 64 logical rows x 128 k: the 128 x 64 source tile goes through LDS so that both the HBM reads (128-byte row segments) and the
// packed writes stay contiguous: lane = (row, 32 k), 4 lanes write 128 consecutive bytes of a row and a wavefront whole blocks.  Bound: HBM.
// PAST: non-temporal loads (reads_past() in kernels.hpp); the stores stay ordinary, two of which make a line (R = 28672, K = 8192: 140 us, non-temporal 179).
//   R = 16384, K = 4096, operands in turn past the last-level cache: 65 us with one row per lane (32 bytes at a row's distance), 47 with four, 43 (4.9 TB/s) with the loads in flight together and
//   the selection on keys; one operand over and over, which that cache serves, 36 and 34; R = 8192, K = 4096 27 and 24, 22 and 20; with the unpruned transpose, R = 28672, K = 8192:
//   296 and 248 us, 234 with the loads in flight together (5.1 TB/s).
template <bool SOFT, bool PAST = false>
__device__ __forceinline__ void prune24_cols_body(void* smem, int bx, int by, int bz, const uint16_t* __restrict__ src, int64_t R, int K, int64_t ld,
                                                          uint16_t* __restrict__ vals, uint8_t* __restrict__ meta,
                                                          uint16_t* __restrict__ vblk, uint8_t* __restrict__ mblk,
                                                          uint16_t* __restrict__ src_t) {
    constexpr int TK = 128, TR = 64, PITCH = TR + 2;
    uint16_t* tile = reinterpret_cast<uint16_t*>(smem);
    (void)TK;
    const int64_t r0 = (int64_t)bx * TR;
    const int k0 = by * TK;
    const int tid = threadIdx.x;
    if (bz) {   // batched form: matrix bz of a stack of [K, R] sources (ld = R)
        const int64_t m = (int64_t)bz * R * K;
        src += m;
        if (vals) { vals += m / 2; meta += m / 8; }
        if (vblk) { vblk += m / 2; mblk += m / 8; }
        if (src_t) src_t += m;
    }
    // all four loads before the first is waited for, so no branch around them: rows past the end, whose results go nowhere, are the last row again
    uint4 w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = k0 + tid / 8 + 32 * i;
        w[i] = load_in<PAST>(src + (int64_t)(k < K ? k : K - 1) * ld + r0 + (tid % 8) * 8);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t* p = reinterpret_cast<uint32_t*>(&tile[(tid / 8 + 32 * i) * PITCH + (tid % 8) * 8]);
        p[0] = w[i].x; p[1] = w[i].y; p[2] = w[i].z; p[3] = w[i].w;
    }
    __syncthreads();
    if (src_t) {        // the unpruned transposed tile: logical rows r (64) x k (128) -> [R, K] row-major, 16 bytes per thread and pass
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // row r0 + tr, k segment of 8 starting at 8 ks: 16 lanes take 256 consecutive bytes of a row
            const int e = tid + 256 * i, tr = e >> 4, ks = e & 15;
            if (k0 + 8 * ks < K) {
                uint32_t o[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o[j] = tile[(8 * ks + 2 * j) * PITCH + tr] | ((uint32_t)tile[(8 * ks + 2 * j + 1) * PITCH + tr] << 16);
                *reinterpret_cast<uint4*>(src_t + (r0 + tr) * K + k0 + 8 * ks) = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    }
    const int rr = tid >> 2, q = tid & 3;
    if (k0 + 32 * q >= K) return;
    uint32_t ov[8], mbytes = 0;
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        const uint16_t* p = &tile[(32 * q + 4 * g) * PITCH + rr];
        uint32_t nib;
        ov[g] = select24<SOFT>(p[0], p[PITCH], p[2 * PITCH], p[3 * PITCH], nib);
        mbytes |= nib << (4 * g);
    }
    const int64_t r = r0 + rr;
    if (vals) {         // (the fused step's lean form passes no canonical outputs: only the blocked copies are consumed)
        uint16_t* vo = vals + r * (K / 2) + (k0 + 32 * q) / 2;
        *reinterpret_cast<uint4*>(vo) = make_uint4(ov[0], ov[1], ov[2], ov[3]);
        *reinterpret_cast<uint4*>(vo + 8) = make_uint4(ov[4], ov[5], ov[6], ov[7]);
        *reinterpret_cast<uint32_t*>(meta + r * (K / 8) + (k0 + 32 * q) / 8) = mbytes;
    }
    if (vblk) {
        uint16_t* vb = vblk + blk_off(r, (k0 + 32 * q) / 2, K / 64);
        *reinterpret_cast<uint4*>(vb) = make_uint4(ov[0], ov[1], ov[2], ov[3]);
        *reinterpret_cast<uint4*>(vb + 8) = make_uint4(ov[4], ov[5], ov[6], ov[7]);
        // 32 k = one step of the matrix instruction: its two 16-k halves belong to different lanes of the unit
        *reinterpret_cast<uint16_t*>(mblk + mblk_off(r, k0 + 32 * q, K / 64)) = (uint16_t)mbytes;
        *reinterpret_cast<uint16_t*>(mblk + mblk_off(r, k0 + 32 * q + 16, K / 64)) = (uint16_t)(mbytes >> 16);
    }
}

// Rows K-contiguous, fused-step variant: a wavefront owns 16 rows x 64 k, i.e. exactly one 1 KB block of the
// blocked packed output; lane = (row, 16 k), two 16-byte loads, one 16-byte store per output.
// logM > 0 (neuron-level experts, Section 3.3): output row e * Kc + j takes source row (j / 4) * M + 4 e + j % 4, i.e.
// the rows of every expert's hidden units come out consecutively (expert-major), ready for one grouped contraction.
template <bool SOFT>
__device__ __forceinline__ void prune24_rows_step_body(int bx, int by, const uint16_t* __restrict__ src, int K, int64_t ld,
                                                               uint16_t* __restrict__ vals, uint8_t* __restrict__ meta,
                                                               uint16_t* __restrict__ vblk, uint8_t* __restrict__ mblk, int logM, int Kc) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunk = bx * 4 + wave;            // 64-k column
    if (chunk * 64 >= K) return;
    const int64_t r = (int64_t)by * 16 + (lane >> 2);
    int64_t rs = r;                                     // source row
    if (logM) { const int e = (int)(r / Kc), j = (int)(r - (int64_t)e * Kc); rs = ((int64_t)(j >> 2) << logM) + 4 * e + (j & 3); }
    const int q = lane & 3, k = chunk * 64 + 16 * q;
    const uint4 w0 = *reinterpret_cast<const uint4*>(src + rs * ld + k);
    const uint4 w1 = *reinterpret_cast<const uint4*>(src + rs * ld + k + 8);
    uint32_t n0, n1, n2, n3;
    const uint32_t o0 = select24<SOFT>(w0.x & 0xFFFFu, w0.x >> 16, w0.y & 0xFFFFu, w0.y >> 16, n0);
    const uint32_t o1 = select24<SOFT>(w0.z & 0xFFFFu, w0.z >> 16, w0.w & 0xFFFFu, w0.w >> 16, n1);
    const uint32_t o2 = select24<SOFT>(w1.x & 0xFFFFu, w1.x >> 16, w1.y & 0xFFFFu, w1.y >> 16, n2);
    const uint32_t o3 = select24<SOFT>(w1.z & 0xFFFFu, w1.z >> 16, w1.w & 0xFFFFu, w1.w >> 16, n3);
    const uint4 ov = make_uint4(o0, o1, o2, o3);
    const uint16_t mb = (uint16_t)(n0 | (n1 << 4) | (n2 << 8) | (n3 << 12));
    if (vals) {
        *reinterpret_cast<uint4*>(vals + r * (K / 2) + k / 2) = ov;
        *reinterpret_cast<uint16_t*>(meta + r * (K / 8) + k / 8) = mb;
    }
    *reinterpret_cast<uint4*>(vblk + blk_off(r, k / 2, K / 64)) = ov;
    *reinterpret_cast<uint16_t*>(mblk + mblk_off(r, k, K / 64)) = mb;
}

}  // namespace sffn
