// prune24_compress: per-iteration 2:4 prune-and-pack of a weight matrix (paper Section 2.2 and the
// "sparsify24" calls of Alg. 1 line 4 / Alg. 2 line 2).  HBM-bound element-wise scan: every input
// element is read once (16-byte loads), 0.5 element of values and 1/16 byte of metadata are written.
#include "common.hpp"
#include "kernels.hpp"
#include "scans.hpp"

namespace sffn {

// ---- rows are K-contiguous: one thread per 8 consecutive elements (two groups) -----------------
template <bool SOFT, bool FLAT, bool PAST>
__global__ void __launch_bounds__(256) prune24_rows_kernel(const uint16_t* __restrict__ src, int64_t nchunks, int cpr,
                                                          int64_t ld, uint16_t* __restrict__ vals,
                                                          uint8_t* __restrict__ meta) {
    constexpr int UNROLL = 4;
    const int64_t base = (int64_t)blockIdx.x * (256 * UNROLL) + threadIdx.x;
    uint4 w[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const int64_t c = base + u * 256;
        if (c < nchunks) {
            int64_t off;
            if (FLAT) off = c * 8;
            else { const int64_t r = c / cpr; off = r * ld + (c - r * cpr) * 8; }
            w[u] = load_in<PAST>(src + off);
        }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const int64_t c = base + u * 256;
        if (c < nchunks) {
            uint32_t n0, n1;
            const uint32_t o0 = select24<SOFT>(w[u].x & 0xFFFFu, w[u].x >> 16, w[u].y & 0xFFFFu, w[u].y >> 16, n0);
            const uint32_t o1 = select24<SOFT>(w[u].z & 0xFFFFu, w[u].z >> 16, w[u].w & 0xFFFFu, w[u].w >> 16, n1);
            if (PAST) __builtin_nontemporal_store((uint64_t)o0 | ((uint64_t)o1 << 32), reinterpret_cast<uint64_t*>(vals + c * 4));
            else *reinterpret_cast<uint2*>(vals + c * 4) = make_uint2(o0, o1);
            meta[c] = (uint8_t)(n0 | (n1 << 4));
        }
    }
}

template <bool SOFT, bool PAST>
__global__ void __launch_bounds__(256) prune24_cols_kernel(const uint16_t* __restrict__ src, int64_t R, int K, int64_t ld, uint16_t* __restrict__ vals,
                                                          uint8_t* __restrict__ meta, uint16_t* __restrict__ vblk, uint8_t* __restrict__ mblk) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kPruneColsLds];
    prune24_cols_body<SOFT, PAST>(smem, blockIdx.x, blockIdx.y, 0, src, R, K, ld, vals, meta, vblk, mblk, nullptr);
}
template <bool SOFT>
__global__ void __launch_bounds__(256) prune24_rows_step_kernel(const uint16_t* __restrict__ src, int K, int64_t ld, uint16_t* __restrict__ vals, uint8_t* __restrict__ meta,
                                                               uint16_t* __restrict__ vblk, uint8_t* __restrict__ mblk, int logM, int Kc) {
    prune24_rows_step_body<SOFT>(blockIdx.x, blockIdx.y, src, K, ld, vals, meta, vblk, mblk, logM, Kc);
}

template <bool SOFT, bool PAST>
static void launch_impl(const uint16_t* src, int64_t R, int64_t K, int64_t ld, int trans, uint16_t* vals, uint8_t* meta, hipStream_t s) {
    const int64_t nchunks = R * (K / 8);
    const dim3 rows((unsigned)((nchunks + 1023) / 1024)), cols((unsigned)(R / 64), (unsigned)((K + 127) / 128));
    if (trans) hipLaunchKernelGGL((prune24_cols_kernel<SOFT, PAST>), cols, dim3(256), 0, s, src, R, (int)K, ld, vals, meta, (uint16_t*)nullptr, (uint8_t*)nullptr);
    else if (ld == K) hipLaunchKernelGGL((prune24_rows_kernel<SOFT, true, PAST>), rows, dim3(256), 0, s, src, nchunks, (int)(K / 8), ld, vals, meta);
    else hipLaunchKernelGGL((prune24_rows_kernel<SOFT, false, PAST>), rows, dim3(256), 0, s, src, nchunks, (int)(K / 8), ld, vals, meta);
}
hipError_t launch_prune24(const uint16_t* src, int64_t R, int64_t K, int64_t ld, int trans, int mode, uint16_t* vals,
                          uint8_t* meta, hipStream_t stream) {
    const bool past = reads_past(2 * R * K);
    if (mode == 0) past ? launch_impl<false, true>(src, R, K, ld, trans, vals, meta, stream) : launch_impl<false, false>(src, R, K, ld, trans, vals, meta, stream);
    else past ? launch_impl<true, true>(src, R, K, ld, trans, vals, meta, stream) : launch_impl<true, false>(src, R, K, ld, trans, vals, meta, stream);
    return hipGetLastError();
}

hipError_t launch_prune24_step(const uint16_t* src, int64_t R, int64_t K, int64_t ld, int trans, int mode, uint16_t* vals,
                               uint8_t* meta, uint16_t* vblk, uint8_t* mblk, hipStream_t stream, int cluster_M) {
    if (cluster_M && (trans || (cluster_M != 8 && cluster_M != 16 && cluster_M != 32 && cluster_M != 64) || R % cluster_M)) return hipErrorInvalidValue;
    if (!trans) {
        dim3 grid((unsigned)((K / 64 + 3) / 4), (unsigned)(R / 16));
        const int logM = cluster_M == 8 ? 3 : cluster_M == 16 ? 4 : cluster_M == 32 ? 5 : cluster_M == 64 ? 6 : 0;
        const int Kc = cluster_M ? (int)(4 * R / cluster_M) : 0;
        if (mode == 0) hipLaunchKernelGGL((prune24_rows_step_kernel<false>), grid, dim3(256), 0, stream, src, (int)K, ld, vals, meta, vblk, mblk, logM, Kc);
        else           hipLaunchKernelGGL((prune24_rows_step_kernel<true>), grid, dim3(256), 0, stream, src, (int)K, ld, vals, meta, vblk, mblk, logM, Kc);
    } else {
        dim3 grid((unsigned)(R / 64), (unsigned)((K + 127) / 128));
        if (mode == 0) hipLaunchKernelGGL((prune24_cols_kernel<false, false>), grid, dim3(256), 0, stream, src, R, (int)K, ld, vals, meta, vblk, mblk);
        else           hipLaunchKernelGGL((prune24_cols_kernel<true, false>), grid, dim3(256), 0, stream, src, R, (int)K, ld, vals, meta, vblk, mblk);
    }
    return hipGetLastError();
}

}  // namespace sffn
