// V:2:M with wider blocks, M in {16, 32, 64} (paper Section 2.3 and Table 5: 64 x M blocks keep 4 columns by L1 score,
// then 2:4 inside them; density 2 / M).  Stand-alone, HBM-bound kernels for the same operations as vnm.hip (M = 8):
// SquaredReLU + compression (eq. (2), Alg. 1 lines 5-6), eq. (6) on the kept slots, the re-expression as a plain 2:4
// matrix over all columns (two survivors per M columns still leave at most two per aligned group of four) and the dense
// transposed expansion for the weight-gradient GEMMs.  Packed layout as for M = 8: vals [T, 2F/M], meta [T, F/(2M)]
// (one nibble per block, two blocks per byte), colidx [T/64, F/M, 4] (offsets inside the block, ascending).
#include "common.hpp"
#include "kernels.hpp"
#include "lds_dma.hpp"
#include "vnm_select.hpp"

namespace sffn {

// One wavefront = one 64-token block x 64 columns (64 / M whole blocks); a workgroup's four stand side by side.  A lane loads 16 bytes of 8 rows, squares
// them and puts them into the wavefront's LDS tile, from which lane = column takes them back, four rows to a transposing read, for the ordered
// fp32 score.  M = 8: the 8 columns a lane has loaded are a block, so the 2:4 choice is made on the registers (the four kept columns come out of them by
// byte permutes that are the same for all rows); M >= 16: on the tile, lane = (row, block).
// 16-byte chunk number seg of row r stands at chunk seg ^ swz(r), and lane group g loads row g ^ (g >> 1) of its eight: the b128 writes, the transposing
// reads and, but for columns that meet by chance, the 2-byte reads then touch every bank once.
// Survivors and metadata of the four wavefronts meet in LDS and leave as whole rows of the workgroup: with every wavefront storing its own 32 and 4 bytes of
// a row, T = F = 16384, M = 8 takes 153 us, with whole rows 124.
//   Bound: HBM.  T = F = 16384: M = 8 147 -> 124 us (0.69 GB, 5.6 TB/s; 111 with the loads past the caches and the rows stored non-temporal), M = 16 135 -> 117, 32 132 -> 115, 64 154 -> 106; T = F = 8192: 35 -> 29, 31 -> 26,
//   33 -> 24, 42 -> 24.  (Before: one 2-byte LDS read per score term, M comparisons per column, ranks out of six comparisons per pair.)  43 KB of LDS, three
//   workgroups per CU: with the survivors in the tile's place four fit, and M = 8 takes 132 us, M = 32 119; two: 31 us at T = F = 8192.
__device__ __forceinline__ uint32_t swz(uint32_t r) { return (((r >> 1) & 1u) << 2) | ((r >> 2) & 1u); }
template <int M, bool PAST>
__global__ void __launch_bounds__(256) sqrelu_vnm_compress_m_kernel(const uint16_t* __restrict__ y1, int64_t F,
                                                                   uint16_t* __restrict__ vals, uint8_t* __restrict__ meta,
                                                                   uint8_t* __restrict__ colidx) {
    constexpr int NB = 64 / M;                           // blocks per wavefront tile
    __shared__ __attribute__((aligned(16))) unsigned char tiles[4][64 * 128];
    __shared__ __attribute__((aligned(16))) unsigned char packed[4][64 * 32];          // [row][block] (of M >= 16 a part is used)
    __shared__ __attribute__((aligned(8))) uint8_t nibs[4][64][NB];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t tb = blockIdx.y;
    const int64_t c0 = (int64_t)blockIdx.x * 256 + wave * 64;
    const bool active = c0 < F;                          // F is a multiple of 64
    unsigned char* tl = tiles[wave];
    if (active) {
        const int seg = lane & 7, r8 = (lane >> 3) ^ (lane >> 4);          // row number of the lane in every eight rows
        uint4 w[8];
        const uint16_t* src = y1 + (tb * 64 + r8) * F + c0 + seg * 8;
#pragma unroll
        for (int it = 0; it < 8; ++it) w[it] = load_in<PAST>(src + it * 8 * F);
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            w[it] = make_uint4(sqrelu2(w[it].x), sqrelu2(w[it].y), sqrelu2(w[it].z), sqrelu2(w[it].w));
            *reinterpret_cast<uint4*>(tl + (it * 8 + r8) * 128 + ((seg ^ swz(r8)) << 4)) = w[it];
        }
        wave_lds_sync();
        // column score: strict ascending-row fp32 sum of y2 (non-negative, so |y2| = y2); a read gives lane = column four rows
        float sc = 0.0f;
        const uint32_t rr = (lane >> 2) & 3u, ch = 2 * (lane >> 4) + ((lane >> 1) & 1u);
#pragma unroll
        for (int r = 0; r < 64; r += 4) {
            const uint32_t at = (r + rr) * 128 + ((ch ^ swz(r + rr)) << 4) + (lane & 1u) * 8;
            const uint2 q = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds_void*)(tl + at)));
            sc = sc + __uint_as_float(q.x << 16);
            sc = sc + __uint_as_float(q.x & 0xFFFF0000u);
            sc = sc + __uint_as_float(q.y << 16);
            sc = sc + __uint_as_float(q.y & 0xFFFF0000u);
        }
        const unsigned long long kept = __ballot(M == 8 ? keep4_of_8(__float_as_uint(sc), lane) : keep4_of<(M > 8 ? M : 16)>(__float_as_uint(sc), lane));
        const int b = lane % NB;                         // the lane's block in the 2:4 choice, and its four kept offsets, ascending, one per byte
        unsigned long long bits = M == 64 ? kept : (kept >> (b * M)) & ((1ull << (M & 63)) - 1ull);
        uint32_t cw = 0;
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            cw |= (uint32_t)__builtin_ctzll(bits) << (8 * n);
            bits &= bits - 1ull;
        }
        if (lane < NB) *reinterpret_cast<uint32_t*>(colidx + (tb * (F / M) + c0 / M + b) * 4) = cw;
        uint32_t v[NB], nib[NB], row[NB];                // of every sweep: survivors, their positions, the lane's row
        if (M == 8) {
            uint32_t sel[4];                             // byte selectors of kept columns (0, 1), (2, 3) among columns 0-3, 4-7
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                sel[2 * p] = sel[2 * p + 1] = 0x0C0C0C0Cu;                  // 0x0C: a zero byte
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint32_t o = (cw >> (8 * (2 * p + e))) & 7u, s2 = 0x0100u + (o & 3u) * 0x0202u, keep = 0xFFFF0000u >> (16 * e);
                    if (o < 4) sel[2 * p] = (sel[2 * p] & keep) | (s2 << (16 * e));
                    else       sel[2 * p + 1] = (sel[2 * p + 1] & keep) | (s2 << (16 * e));
                }
            }
#pragma unroll
            for (int it = 0; it < NB; ++it) {
                const uint32_t y01 = __builtin_amdgcn_perm(w[it].y, w[it].x, sel[0]) | __builtin_amdgcn_perm(w[it].w, w[it].z, sel[1]);
                const uint32_t y23 = __builtin_amdgcn_perm(w[it].y, w[it].x, sel[2]) | __builtin_amdgcn_perm(w[it].w, w[it].z, sel[3]);
                uint32_t low, high;
                row[it] = it * 8 + r8;
                v[it] = pick24_pos(y01, y23, {3u, 2u, 1u, 0u}, low, high);
                nib[it] = ((low & 3u) | ((high & 3u) << 2)) ^ 0xFu;
            }
        } else {
            const uint32_t q0 = (b * M + (cw & 0xFFu)) * 2, q1 = (b * M + ((cw >> 8) & 0xFFu)) * 2, q2 = (b * M + ((cw >> 16) & 0xFFu)) * 2, q3 = (b * M + (cw >> 24)) * 2;
#pragma unroll
            for (int it = 0; it < NB; ++it) {
                row[it] = it * M + lane / NB;
                const uint32_t x = swz(row[it]) << 4;
                const unsigned char* rp = tl + row[it] * 128;
                const uint32_t y01 = *reinterpret_cast<const uint16_t*>(rp + (q0 ^ x)) | ((uint32_t)*reinterpret_cast<const uint16_t*>(rp + (q1 ^ x)) << 16);
                const uint32_t y23 = *reinterpret_cast<const uint16_t*>(rp + (q2 ^ x)) | ((uint32_t)*reinterpret_cast<const uint16_t*>(rp + (q3 ^ x)) << 16);
                uint32_t low, high;
                v[it] = pick24_pos(y01, y23, {3u, 2u, 1u, 0u}, low, high);
                nib[it] = ((low & 3u) | ((high & 3u) << 2)) ^ 0xFu;
            }
        }
        const uint32_t flip = M == 8 ? (wave & 1) << 7 : 0;      // (the reads below then meet every bank once)
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            *reinterpret_cast<uint32_t*>(packed[wave] + (((row[it] * NB + b) * 4) ^ flip)) = v[it];
            nibs[wave][row[it]][b] = (uint8_t)nib[it];
        }
    }
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * 256;
    constexpr int LANES = M == 8 ? 8 : 4 * NB;           // lanes that write the 4 NB words of a row
#pragma unroll
    for (int i = 0; i < 64 * LANES / 256; ++i) {
        const int e = threadIdx.x + 256 * i, row = e / LANES, j = e % LANES;
        if (M == 8) {
            if (b0 + j * 32 < F) {
                const uint4 w = *reinterpret_cast<const uint4*>(packed[j >> 1] + ((row * 32 + (j & 1) * 16) ^ ((j & 2) << 6)));
                uint16_t* const p = vals + (tb * 64 + row) * (F / 4) + b0 / 4 + j * 8;
                if (PAST) store_out(p, w); else *reinterpret_cast<uint4*>(p) = w;
            }
        } else if (b0 + j * M < F) {
            *reinterpret_cast<uint32_t*>(vals + (tb * 64 + row) * (2 * F / M) + (b0 / M + j) * 2) = *reinterpret_cast<const uint32_t*>(packed[j / NB] + (row * NB + j % NB) * 4);
        }
    }
    // metadata: lane = (row, the 32 / M bytes of a wavefront); M = 64: a byte belongs to two wavefronts
    const int row = threadIdx.x >> 2, j = threadIdx.x & 3;
    if (b0 + 64 * j < F) {
        uint8_t* mp = meta + (tb * 64 + row) * (F / (2 * M)) + (b0 + 64 * j) / (2 * M);
        if (M == 8) {
            const uint2 n = *reinterpret_cast<const uint2*>(nibs[j][row]);
            *reinterpret_cast<uint32_t*>(mp) = __builtin_amdgcn_perm(n.y | (n.y >> 4), n.x | (n.x >> 4), 0x06040200u);
        } else if (M == 16) {
            const uint32_t n = *reinterpret_cast<const uint32_t*>(nibs[j][row]), z = n | (n >> 4);
            *reinterpret_cast<uint16_t*>(mp) = (uint16_t)((z & 0xFFu) | ((z >> 8) & 0xFF00u));
        } else if (M == 32) {
            *mp = (uint8_t)(nibs[j][row][0] | (nibs[j][row][NB - 1] << 4));
        } else if (!(j & 1)) {
            *mp = (uint8_t)(nibs[j][row][0] | (nibs[j + 1][row][0] << 4));
        }
    }
}

// eq. (6) on y2's kept slots; one thread per (token, block).
__global__ void __launch_bounds__(256) dsqrelu_vnm_m_kernel(const uint16_t* __restrict__ dy2, const uint16_t* __restrict__ y1,
                                                           const uint8_t* __restrict__ meta, const uint8_t* __restrict__ colidx,
                                                           int64_t F, int M, int nblk, uint16_t* __restrict__ dvals) {
    const int blk = blockIdx.x * 256 + threadIdx.x;
    if (blk >= nblk) return;
    const int64_t t = blockIdx.y;
    const uint32_t cw = *reinterpret_cast<const uint32_t*>(colidx + ((t >> 6) * nblk + blk) * 4);
    const uint32_t nib = (meta[t * (nblk / 2) + (blk >> 1)] >> (4 * (blk & 1))) & 0xFu;
    const uint32_t o0 = (cw >> (8 * (nib & 3u))) & 0xFFu, o1 = (cw >> (8 * (nib >> 2))) & 0xFFu;
    const int64_t base = t * F + (int64_t)blk * M;
    const float ya = bf2f(y1[base + o0]), yb = bf2f(y1[base + o1]);
    const float ga = 2.0f * bf2f(dy2[base + o0]) * (ya > 0.0f ? ya : 0.0f);
    const float gb = 2.0f * bf2f(dy2[base + o1]) * (yb > 0.0f ? yb : 0.0f);
    *reinterpret_cast<uint32_t*>(dvals + t * (2 * (int64_t)nblk) + (int64_t)blk * 2) = f2bf2(ga, gb);
}

// The V:2:M matrix as a plain 2:4 matrix over all F columns: vals24 [T, F/2], meta24 [T, F/8] (row-major).  One thread
// per (token, block) writes the block's M / 4 groups; a group holds both survivors, one (next to an empty slot) or none.
__global__ void __launch_bounds__(256) vnm_to_24_m_kernel(const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                                                         const uint8_t* __restrict__ colidx, int64_t F, int M, int nblk,
                                                         uint16_t* __restrict__ vals24, uint8_t* __restrict__ meta24) {
    const int blk = blockIdx.x * 256 + threadIdx.x;
    if (blk >= nblk) return;
    const int64_t t = blockIdx.y;
    const uint32_t cw = *reinterpret_cast<const uint32_t*>(colidx + ((t >> 6) * nblk + blk) * 4);
    const uint32_t nib = (meta[t * (nblk / 2) + (blk >> 1)] >> (4 * (blk & 1))) & 0xFu;
    const uint32_t v = *reinterpret_cast<const uint32_t*>(vals + t * (2 * (int64_t)nblk) + (int64_t)blk * 2);
    const uint32_t o0 = (cw >> (8 * (nib & 3u))) & 0xFFu, o1 = (cw >> (8 * (nib >> 2))) & 0xFFu;    // o0 < o1
    const uint32_t v0 = v & 0xFFFFu, v1 = v >> 16;
    uint32_t* vo = reinterpret_cast<uint32_t*>(vals24 + t * (F / 2) + (int64_t)blk * (M / 2));
    uint8_t* mo = meta24 + t * (F / 8) + (int64_t)blk * (M / 8);
    uint32_t prev = 0;
    for (int g = 0; g < M / 4; ++g) {
        const bool in0 = (o0 >> 2) == (uint32_t)g, in1 = (o1 >> 2) == (uint32_t)g;
        const uint32_t p = o0 & 3u, q = o1 & 3u;
        uint32_t a = 0, n = 0x4u;                                   // empty group: +0 at positions 0, 1
        if (in0 && in1) { a = v; n = p | (q << 2); }
        else if (in0)   { a = (p < 3) ? v0 : (v0 << 16); n = (p < 3) ? (p | (3u << 2)) : (3u << 2); }
        else if (in1)   { a = (q > 0) ? (v1 << 16) : v1; n = (q > 0) ? (q << 2) : 0x4u; }
        vo[g] = a;
        if (g & 1) mo[g >> 1] = (uint8_t)(prev | (n << 4)); else prev = n;
    }
}

// Dense transposed expansion AT[f, t] (row-major [F, T]); one workgroup = 64 tokens x 64 columns through LDS.
__global__ void __launch_bounds__(256) vnm_expand_t_m_kernel(const uint16_t* __restrict__ vals, const uint8_t* __restrict__ meta,
                                                            const uint8_t* __restrict__ colidx, int64_t T, int64_t F, int M,
                                                            int nblk, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[64][64 + 8];
    const int tid = threadIdx.x;
    for (int i = tid; i < 64 * 72 / 2; i += 256) reinterpret_cast<uint32_t*>(&tile[0][0])[i] = 0;
    __syncthreads();
    const int64_t tb = blockIdx.y;
    const int nb = 64 / M, b0 = blockIdx.x * nb;                   // first block of this 64-column tile
    for (int e = tid; e < 64 * nb; e += 256) {
        const int r = e / nb, bl = e % nb, blk = b0 + bl;
        const int64_t t = tb * 64 + r;
        const uint32_t cw = *reinterpret_cast<const uint32_t*>(colidx + (tb * nblk + blk) * 4);
        const uint32_t nib = (meta[t * (nblk / 2) + (blk >> 1)] >> (4 * (blk & 1))) & 0xFu;
        const uint32_t o0 = (cw >> (8 * (nib & 3u))) & 0xFFu, o1 = (cw >> (8 * (nib >> 2))) & 0xFFu;
        const uint32_t v = *reinterpret_cast<const uint32_t*>(vals + t * (2 * (int64_t)nblk) + (int64_t)blk * 2);
        tile[bl * M + o0][r] = (uint16_t)(v & 0xFFFFu);
        tile[bl * M + o1][r] = (uint16_t)(v >> 16);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = tid + 256 * i, fr = e >> 3, seg = e & 7;     // 64 rows x 8 segments of 8 tokens
        *reinterpret_cast<uint4*>(out + ((int64_t)blockIdx.x * 64 + fr) * T + tb * 64 + seg * 8) = *reinterpret_cast<const uint4*>(&tile[fr][seg * 8]);
    }
}

template <int M>
static void launch_compress(const uint16_t* y1, int64_t T, int64_t F, uint16_t* vals, uint8_t* meta, uint8_t* colidx, hipStream_t s) {
    const dim3 grid((unsigned)((F + 255) / 256), (unsigned)(T / 64));
    if (reads_past(2 * T * F)) hipLaunchKernelGGL((sqrelu_vnm_compress_m_kernel<M, true>), grid, dim3(256), 0, s, y1, F, vals, meta, colidx);
    else hipLaunchKernelGGL((sqrelu_vnm_compress_m_kernel<M, false>), grid, dim3(256), 0, s, y1, F, vals, meta, colidx);
}
hipError_t launch_sqrelu_vnm_compress_m(const uint16_t* y1, int64_t T, int64_t F, int M, uint16_t* vals, uint8_t* meta, uint8_t* colidx,
                                        hipStream_t s) {
    if (M == 8)       launch_compress<8>(y1, T, F, vals, meta, colidx, s);
    else if (M == 16) launch_compress<16>(y1, T, F, vals, meta, colidx, s);
    else if (M == 32) launch_compress<32>(y1, T, F, vals, meta, colidx, s);
    else if (M == 64) launch_compress<64>(y1, T, F, vals, meta, colidx, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_dsqrelu_vnm_m(const uint16_t* dy2, const uint16_t* y1, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F,
                                int M, uint16_t* dvals, hipStream_t s) {
    const int nblk = (int)(F / M);
    dim3 grid((unsigned)((nblk + 255) / 256), (unsigned)T);
    hipLaunchKernelGGL(dsqrelu_vnm_m_kernel, grid, dim3(256), 0, s, dy2, y1, meta, colidx, F, M, nblk, dvals);
    return hipGetLastError();
}

hipError_t launch_vnm_to_24_m(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M,
                              uint16_t* vals24, uint8_t* meta24, hipStream_t s) {
    const int nblk = (int)(F / M);
    dim3 grid((unsigned)((nblk + 255) / 256), (unsigned)T);
    hipLaunchKernelGGL(vnm_to_24_m_kernel, grid, dim3(256), 0, s, vals, meta, colidx, F, M, nblk, vals24, meta24);
    return hipGetLastError();
}

hipError_t launch_vnm_expand_t_m(const uint16_t* vals, const uint8_t* meta, const uint8_t* colidx, int64_t T, int64_t F, int M,
                                 uint16_t* out, hipStream_t s) {
    const int nblk = (int)(F / M);
    dim3 grid((unsigned)(F / 64), (unsigned)(T / 64));
    hipLaunchKernelGGL(vnm_expand_t_m_kernel, grid, dim3(256), 0, s, vals, meta, colidx, T, F, M, nblk, out);
    return hipGetLastError();
}

}  // namespace sffn
