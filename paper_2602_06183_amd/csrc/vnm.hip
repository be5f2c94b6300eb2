// V:N:M (V=64, N=2, M=8) kernels: eq. (6) on the kept slots (Alg. 2 line 4) and the layout helpers the GEMMs
// consume (re-expression as plain 2:4 over all columns, dense transposed expansion, bf16 transpose).  All of them
// are HBM-bound scans.  The stand-alone compressor of eq. (2) + Section 2.3 lives in vnm_general.hip, for every M.
#include "common.hpp"
#include "kernels.hpp"
#include "scans.hpp"

namespace sffn {

__device__ __forceinline__ uint32_t pick16(const uint32_t (&w)[4], uint32_t c) {
    const uint32_t d = c >> 1;
    const uint32_t lo = (d == 0) ? w[0] : (d == 1) ? w[1] : (d == 2) ? w[2] : w[3];
    return (c & 1u) ? (lo >> 16) : (lo & 0xFFFFu);
}

// eq. (6) evaluated only where y2 was kept.  One thread per (row, column block).
//   Bound: HBM.  T = F = 16384, 1.2 GB: 213 us, 197 (6.2 TB/s) past the caches; four rows a thread 196, eight 200.
template <bool PAST>
__global__ void __launch_bounds__(256) dsqrelu_vnm_kernel(const uint16_t* __restrict__ dy2, const uint16_t* __restrict__ y1,
                                                         const uint8_t* __restrict__ meta, const uint8_t* __restrict__ colidx,
                                                         int64_t F, int nblk, uint16_t* __restrict__ dvals) {
    const int blk = blockIdx.x * 256 + threadIdx.x;
    if (blk >= nblk) return;          // nblk is a multiple of 8, so groups of 4 lanes are in or out together
    const int64_t t = blockIdx.y;
    const uint32_t cw = *reinterpret_cast<const uint32_t*>(colidx + ((t >> 6) * nblk + blk) * 4);
    const uint32_t nib = (meta[t * (F / 16) + (blk >> 1)] >> (4 * (blk & 1))) & 0xFu;
    const uint32_t o0 = (cw >> (8 * (nib & 3u))) & 0xFFu, o1 = (cw >> (8 * (nib >> 2))) & 0xFFu;
    const uint4 d4 = load_in<PAST>(dy2 + t * F + (int64_t)blk * 8);
    const uint4 y4 = load_in<PAST>(y1 + t * F + (int64_t)blk * 8);
    const uint32_t dw[4] = {d4.x, d4.y, d4.z, d4.w}, yw[4] = {y4.x, y4.y, y4.z, y4.w};
    const float ya = bf2f(pick16(yw, o0)), yb = bf2f(pick16(yw, o1));
    const float ga = 2.0f * bf2f(pick16(dw, o0)) * (ya > 0.0f ? ya : 0.0f);
    const float gb = 2.0f * bf2f(pick16(dw, o1)) * (yb > 0.0f ? yb : 0.0f);
    const uint32_t v = f2bf2(ga, gb);
    *reinterpret_cast<uint32_t*>(dvals + t * (F / 4) + (int64_t)blk * 2) = v;
}

// Two survivors per 8 columns leave at most two per aligned group of four, so a V:2:8 matrix is
// also a plain 2:4 matrix over all F columns.  This writes that view: vals24 [T, F/2], meta24
// [T, F/8] in the 2:4 packed format (empty slots are +0 at unused positions).
__global__ void __launch_bounds__(256) vnm_to_24_kernel(const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                                                       const uint8_t* __restrict__ colidx, int64_t F, int nblk,
                                                       uint16_t* __restrict__ vals24, uint8_t* __restrict__ meta24) {
    const int blk = blockIdx.x * 256 + threadIdx.x;
    if (blk >= nblk) return;
    const int64_t t = blockIdx.y;
    const uint32_t cw = *reinterpret_cast<const uint32_t*>(colidx + ((t >> 6) * nblk + blk) * 4);
    const uint32_t nib = (meta[t * (F / 16) + (blk >> 1)] >> (4 * (blk & 1))) & 0xFu;
    const uint32_t v = *reinterpret_cast<const uint32_t*>(vals + t * (F / 4) + (int64_t)blk * 2);
    uint32_t a, b, mb;
    vnm_block_to_24(v, nib, cw, a, b, mb);
    *reinterpret_cast<uint2*>(vals24 + t * (F / 2) + (int64_t)blk * 4) = make_uint2(a, b);
    meta24[t * (F / 8) + blk] = (uint8_t)mb;
}

// The transposed operand of the weight-gradient contractions from the canonical arrays, as the fused epilogues write it: KEPT = false: at = the
// survivors compacted to 4 rows per 8 hidden units (gemm_wgrad_body.hpp), [F / 2, T] blocked, and mask = the kept-column bits of every 8;
// KEPT = true (M = 32, 64): the 4 kept rows of every block in the order of gemm_wgrad_wide_body.hpp.
// One workgroup = 64 tokens x 256 (KEPT: 16 M) hidden units through LDS: rows of 128 bytes at M = 8 in, whole 1 KB blocks out.
//   Bound: HBM.  T = F = 8192, M = 8: 42 MB in, 67 MB out: 29 us; the dense [F, T] expansion took 51 us.
constexpr int kCompactRows = 128, kCompactPitch = 64 + 2, kCompactLds = kCompactRows * kCompactPitch * 2 + 32 * 4 + 32;
template <bool KEPT>
__device__ __forceinline__ void vnm_compact_t_body(void* smem, int bx, int64_t tb, const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                                                   const uint8_t* __restrict__ colidx, int64_t T, int64_t F, int logM, uint16_t* __restrict__ at, uint8_t* __restrict__ mask) {
    constexpr int ROWS = KEPT ? 64 : kCompactRows, PITCH = kCompactPitch;
    uint32_t* const tile32 = reinterpret_cast<uint32_t*>(smem);
    uint32_t* const cols = tile32 + kCompactRows * PITCH / 2;              // kept columns of the workgroup's blocks
    uint8_t* const gm = reinterpret_cast<uint8_t*>(cols + 32);             // and, as bits, of its groups of 8 hidden units
    uint16_t* const tile = reinterpret_cast<uint16_t*>(tile32);
    const int tid = threadIdx.x;
    const int64_t nblk = F >> logM;
    const int lognb = KEPT ? 4 : 8 - logM, nb = 1 << lognb;              // blocks of the workgroup
    const int64_t b0 = (int64_t)bx << lognb;
    const int here = nblk - b0 < nb ? (int)(nblk - b0) : nb;
    for (int i = tid; i < ROWS * PITCH / 2; i += 256) tile32[i] = 0;
    if (!KEPT && tid < here) cols[tid] = *reinterpret_cast<const uint32_t*>(colidx + (tb * nblk + b0 + tid) * 4);
    __syncthreads();
    if (!KEPT) {
        if (tid < here << (logM - 3)) {            // a group of 8 hidden units: which of them are among its block's kept columns
            const uint32_t c = cols[tid >> (logM - 3)], g = tid & ((1 << (logM - 3)) - 1);
            uint32_t m = 0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t o = (c >> (8 * p)) & 0xFFu;
                m |= (o >> 3) == g ? 1u << (o & 7) : 0u;
            }
            gm[tid] = (uint8_t)m;
            mask[tb * (F >> 3) + (b0 << (logM - 3)) + tid] = (uint8_t)m;
        }
        __syncthreads();
    }
    for (int e = tid; e < 64 << lognb; e += 256) {
        const int r = e >> lognb, bl = e & (nb - 1);
        if (bl >= here) continue;
        const int64_t t = tb * 64 + r, blk = b0 + bl;
        const uint32_t nib = (meta[t * (nblk >> 1) + (blk >> 1)] >> (4 * (blk & 1))) & 0xFu;
        const uint32_t v = *reinterpret_cast<const uint32_t*>(vals + t * (2 * nblk) + blk * 2);
        const uint32_t p0 = nib & 3u, p1 = nib >> 2;
        int r0 = bl * 4 + p0, r1 = bl * 4 + p1;
        if (!KEPT) {
            const uint32_t o0 = (cols[bl] >> (8 * p0)) & 0xFFu, o1 = (cols[bl] >> (8 * p1)) & 0xFFu;
            const int g0 = (bl << (logM - 3)) + (o0 >> 3), g1 = (bl << (logM - 3)) + (o1 >> 3);
            r0 = g0 * 4 + __builtin_popcount(gm[g0] & ((1u << (o0 & 7)) - 1u));
            r1 = g1 * 4 + __builtin_popcount(gm[g1] & ((1u << (o1 & 7)) - 1u));
        }
        tile[r0 * PITCH + r] = (uint16_t)(v & 0xFFFFu);
        tile[r1 * PITCH + r] = (uint16_t)(v >> 16);
    }
    __syncthreads();
    const int64_t row0 = KEPT ? b0 * 4 : b0 << (logM - 1), rows = KEPT ? nblk * 4 : F >> 1;
#pragma unroll
    for (int i = 0; i < ROWS / 32; ++i) {
        const int e = tid + 256 * i, l = e & 63;
        const int fr = KEPT ? (e >> 8) * 32 + (e & 31) : (e >> 7) * 16 + (l >> 2);
        const int tc = KEPT ? ((e >> 6) & 3) * 16 + ((e >> 5) & 1) * 8 : ((e >> 6) & 1) * 32 + (l & 3) * 8;
        if (row0 + fr >= rows) continue;
        const uint32_t* p = tile32 + (fr * PITCH + tc) / 2;
        *reinterpret_cast<uint4*>(at + (KEPT ? kept_off(row0 + fr, tb * 64 + tc, rows >> 5) : blk_off(row0 + fr, tb * 64 + tc, T / 32))) = make_uint4(p[0], p[1], p[2], p[3]);
    }
}

__global__ void __launch_bounds__(256) transpose_bf16_kernel(const uint16_t* __restrict__ in, int64_t R, int64_t C, int64_t ld,
                                                            uint16_t* __restrict__ out, int blocked, uint16_t* __restrict__ out_same, unsigned* __restrict__ counters) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kTransposeLds];
    if (counters && blockIdx.x == 0 && blockIdx.y == 0) for (int k = threadIdx.x; k < kSplitCounters; k += 256) counters[k] = 0;
    transpose_bf16_body(smem, blockIdx.x, blockIdx.y, in, R, C, ld, out, blocked, out_same, nullptr);
}

hipError_t launch_dsqrelu_vnm(const uint16_t* dy2, const uint16_t* y1, const uint8_t* meta, const uint8_t* colidx, int64_t T,
                              int64_t F, uint16_t* dvals, hipStream_t s) {
    const int nblk = (int)(F / 8);
    dim3 grid((unsigned)((nblk + 255) / 256), (unsigned)T);
    if (reads_past(4 * T * F)) hipLaunchKernelGGL((dsqrelu_vnm_kernel<true>), grid, dim3(256), 0, s, dy2, y1, meta, colidx, F, nblk, dvals);
    else hipLaunchKernelGGL((dsqrelu_vnm_kernel<false>), grid, dim3(256), 0, s, dy2, y1, meta, colidx, F, nblk, dvals);
    return hipGetLastError();
}

// The canonical V:2:8 arrays regrouped into the units of the V:2:8 activation GEMM (gemm_vnm8.hip; the fused epilogues write them directly).
// One workgroup = 64 tokens x 512 hidden units: a wavefront reads 256 bytes of each of 4 tokens and writes 128 bytes of each of 8 units.
//   Bound: HBM.  T = F = 8192: 75 MB in all; 44 us when every lane moved 32 bytes of a unit of its own, 16 us now.
__device__ __forceinline__ void vnm8_repack_body(int bx, int64_t tb, const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                                                 const uint8_t* __restrict__ colidx, int64_t T, int F, uint16_t* __restrict__ vcb,
                                                 uint8_t* __restrict__ mcb, uint8_t* __restrict__ cixt) {
    const int KS = F >> 6, tid = threadIdx.x, kt0 = bx * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) {                      // 64 tokens x 8 units x two 16-byte halves
        const int e = tid + 256 * i, half = e & 1, kt = kt0 + ((e >> 1) & 7);
        const int64_t t = tb * 64 + (e >> 4);
        if (kt < KS)
            *reinterpret_cast<uint4*>(vcb + vcb_off(t, (int64_t)kt * 8, F) + half * 8) = *reinterpret_cast<const uint4*>(vals + t * (F >> 2) + kt * 16 + half * 8);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 256 * i, kt = kt0 + (e & 7);
        const int64_t t = tb * 64 + (e >> 3);
        if (kt < KS) *reinterpret_cast<uint32_t*>(mcb + mcb_off(t, kt, F)) = *reinterpret_cast<const uint32_t*>(meta + t * (F >> 4) + kt * 4);
    }
    const int kt = kt0 + (tid >> 3), q = tid & 7;
    if (tid < 64 && kt < KS) {        // word (h, r), byte j = kept column r of column block 4 (j / 2) + j % 2 + 2 h
        const int h = q >> 2, r = q & 3;
        const uint8_t* c = colidx + (tb * (F >> 3) + kt * 8) * 4;
        uint32_t dw = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) dw |= (uint32_t)c[(4 * (j >> 1) + (j & 1) + 2 * h) * 4 + r] << (8 * j);
        *reinterpret_cast<uint32_t*>(cixt + cixt_off(tb, kt, T >> 6) + q * 4) = dw;
    }
}

// Both passes come with the transpose of the contraction's other operand, in one launch (on small shapes a launch of its own costs as much as the
// pass): workgroups past the first nc x n_tb tiles take 64 x 64 tiles of it, tc per 64 rows.
struct TransposeOf { const uint16_t* in; int64_t R, C, ld; uint16_t* out; int layout, tc; };
__device__ __forceinline__ void transpose_part(void* smem, int i, const TransposeOf& t) {
    transpose_bf16_body(smem, i % t.tc, i / t.tc, t.in, t.R, t.C, t.ld, t.out, t.layout, nullptr, nullptr);
}
__global__ void __launch_bounds__(256) vnm8_repack_kernel(const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta, const uint8_t* __restrict__ colidx, int64_t T,
                                                         int F, uint16_t* __restrict__ vcb, uint8_t* __restrict__ mcb, uint8_t* __restrict__ cixt, int nc, int n_own, TransposeOf t, unsigned* __restrict__ counters) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kTransposeLds];
    const int i = blockIdx.x;
    if (i == 0 && counters) for (int k = threadIdx.x; k < kSplitCounters; k += 256) counters[k] = 0;
    if (i < n_own) vnm8_repack_body(i % nc, i / nc, vals, meta, colidx, T, F, vcb, mcb, cixt);
    else transpose_part(smem, i - n_own, t);
}
template <bool KEPT>
__global__ void __launch_bounds__(256) vnm_compact_t_kernel(const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta, const uint8_t* __restrict__ colidx, int64_t T,
                                                           int64_t F, int logM, uint16_t* __restrict__ at, uint8_t* __restrict__ mask, int nc, int n_own, TransposeOf t) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kCompactLds];
    static_assert(kCompactLds >= kTransposeLds, "either part");
    const int i = blockIdx.x;
    if (i < n_own) vnm_compact_t_body<KEPT>(smem, i % nc, i / nc, vals, meta, colidx, T, F, logM, at, mask);
    else transpose_part(smem, i - n_own, t);
}
static int64_t transpose_tiles(TransposeOf* t) { t->tc = (int)(t->C / 64); return t->in ? t->C / 64 * (t->R / 64) : 0; }

hipError_t launch_vnm8_repack(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, uint16_t* vcb, uint8_t* mcb,
                              uint8_t* cixt, const uint16_t* W, int64_t R, int64_t C, int64_t ld, uint16_t* wt, unsigned* counters, hipStream_t s) {
    TransposeOf t = {W, R, C, ld, wt, 0, 0};
    const int64_t nc = (F + 511) / 512, own = nc * (T / 64), n = own + transpose_tiles(&t);
    if (n >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(vnm8_repack_kernel, dim3((unsigned)n), dim3(256), 0, s, vals, meta, colidx, T, (int)F, vcb, mcb, cixt, (int)nc, (int)own, t, counters);
    return hipGetLastError();
}

hipError_t launch_vnm_to_24(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F,
                            uint16_t* vals24, uint8_t* meta24, hipStream_t s) {
    const int nblk = (int)(F / 8);
    dim3 grid((unsigned)((nblk + 255) / 256), (unsigned)T);
    hipLaunchKernelGGL(vnm_to_24_kernel, grid, dim3(256), 0, s, vals, meta, colidx, F, nblk, vals24, meta24);
    return hipGetLastError();
}

hipError_t launch_vnm_compact_t(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M, int kept, uint16_t* at,
                                uint8_t* mask, const uint16_t* G, int64_t N, uint16_t* gt, hipStream_t s) {
    const int logM = M == 8 ? 3 : M == 16 ? 4 : M == 32 ? 5 : M == 64 ? 6 : 0;
    if (!logM || (kept && F % (8 * M))) return hipErrorInvalidValue;
    TransposeOf t = {G, T, N, N, gt, kept ? 2 : 1, 0};
    const int64_t width = kept ? 16 * M : 256, nc = (F + width - 1) / width, own = nc * (T / 64), n = own + transpose_tiles(&t);
    if (n >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    if (kept) hipLaunchKernelGGL(vnm_compact_t_kernel<true>, dim3((unsigned)n), dim3(256), 0, s, vals, meta, colidx, T, F, logM, at, mask, (int)nc, (int)own, t);
    else hipLaunchKernelGGL(vnm_compact_t_kernel<false>, dim3((unsigned)n), dim3(256), 0, s, vals, meta, colidx, T, F, logM, at, mask, (int)nc, (int)own, t);
    return hipGetLastError();
}

hipError_t launch_transpose(const uint16_t* in, int64_t R, int64_t C, int64_t ld, uint16_t* out, int blocked, uint16_t* out_same, hipStream_t s, unsigned* counters) {
    dim3 grid((unsigned)(C / 64), (unsigned)(R / 64));
    hipLaunchKernelGGL(transpose_bf16_kernel, grid, dim3(256), 0, s, in, R, C, ld, out, blocked, out_same, counters);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256) clear_counters_kernel(unsigned* counters) { counters[blockIdx.x * 256 + threadIdx.x] = 0; }
hipError_t launch_clear_counters(unsigned* counters, hipStream_t s) {
    hipLaunchKernelGGL(clear_counters_kernel, dim3(kSplitCounters / 256), dim3(256), 0, s, counters);
    return hipGetLastError();
}

}  // namespace sffn
