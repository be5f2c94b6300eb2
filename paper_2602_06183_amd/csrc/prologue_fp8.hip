// The passes of the fp8 step that only depend on its inputs, as one launch or, for large inputs, three: X and dY as codes in their own orientation
// (eqs. (1), (4)) and transposed as codes or bf16 (eqs. (8), (5)); W1 and W2.T pruned and packed as blocked codes (eqs. (1), (4)) and, unpruned, as
// row-major codes (eqs. (7), (3)).  All outputs in the layouts of common.hpp, a pair of codes per 2-byte element.
//   Bound: HBM; every input is read once and every store of a wavefront covers whole blocks or 128-byte rows.
// Every part also records the largest magnitude of its input, one float per workgroup (no atomics and nothing to clear first), and the parts over X
// and dY clear the slots that the epilogues of eqs. (1), (4) collect into.
#include "amax_fold.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace sffn {

namespace {

__device__ __forceinline__ float mag8(float m, const uint4& w) {
    const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) m = __builtin_fmaxf(m, __builtin_fmaxf(bf2f(v[k] & 0x7FFFu), bf2f((v[k] >> 16) & 0x7FFFu)));
    return m;
}
__device__ __forceinline__ uint2 enc8(const uint4& w, float inv) {
    return make_uint2(fp8_enc2(bf2f(w.x & 0xFFFFu), bf2f(w.x >> 16), inv) | (fp8_enc2(bf2f(w.y & 0xFFFFu), bf2f(w.y >> 16), inv) << 16),
                      fp8_enc2(bf2f(w.z & 0xFFFFu), bf2f(w.z >> 16), inv) | (fp8_enc2(bf2f(w.w & 0xFFFFu), bf2f(w.w >> 16), inv) << 16));
}
// one float per workgroup; part = LDS that nothing else uses
__device__ __forceinline__ void note_part(float* out, float m, float* part) {
    if (!out) return;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) *out = __builtin_fmaxf(__builtin_fmaxf(part[0], part[1]), __builtin_fmaxf(part[2], part[3]));
}

constexpr int kTransP = 64 + 2, kColsP = 64 + 2, kLds = 128 * kColsP * 2;

// [R, C] -> codes, blocked, and the transpose as codes (CODES) or bf16, blocked; a 64 x 64 tile
__device__ __forceinline__ void quantize_body(unsigned char* smem, int bx, int by, const uint16_t* __restrict__ src, int64_t R, int64_t C, float inv, bool codes,
                                              uint16_t* __restrict__ out_t, uint16_t* __restrict__ out_same, float* amax, float* part) {
    uint16_t* const tile = reinterpret_cast<uint16_t*>(smem);
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)by * 64, c0 = (int64_t)bx * 64;
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = tid / 8 + 32 * i, seg = tid % 8;
        const uint4 w = *reinterpret_cast<const uint4*>(src + (r0 + r) * C + c0 + seg * 8);
        uint32_t* d = reinterpret_cast<uint32_t*>(&tile[r * kTransP + seg * 8]);
        d[0] = w.x; d[1] = w.y; d[2] = w.z; d[3] = w.w;
        m = mag8(m, w);
        *reinterpret_cast<uint2*>(out_same + blk_off(r0 + r, (c0 + seg * 8) / 2, C / 64)) = enc8(w, inv);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int c = tid / 8 + 32 * i, rs = (tid % 8) * 8;          // output row c0 + c, its 8 elements for source rows r0 + rs .. + 7
        if (!codes) { const int e = tid + 256 * i, bk = e >> 6, l = e & 63; c = (bk >> 1) * 16 + (l >> 2); rs = (bk & 1) * 32 + (l & 3) * 8; }
        uint32_t q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = tile[(rs + 2 * j) * kTransP + c] | ((uint32_t)tile[(rs + 2 * j + 1) * kTransP + c] << 16);
        const uint4 w = make_uint4(q[0], q[1], q[2], q[3]);
        if (codes) *reinterpret_cast<uint2*>(out_t + blk_off(c0 + c, (r0 + rs) / 2, R / 64)) = enc8(w, inv);
        else       *reinterpret_cast<uint4*>(out_t + blk_off(c0 + c, r0 + rs, R / 32)) = w;
    }
    note_part(amax, m, part);
}

// groups along K; a wavefront takes 16 rows x 128 k, one block of packed codes, in four loads of 4 rows x 256 bytes
template <bool SOFT>
__device__ __forceinline__ void prune_rows_body(int bx, int by, const uint16_t* __restrict__ src, int K, float inv, uint8_t* __restrict__ codes, uint8_t* __restrict__ meta,
                                                uint16_t* __restrict__ codes_blk, uint8_t* __restrict__ meta_blk, uint8_t* __restrict__ s_q, float* amax, float* part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k0 = (bx * 4 + wave) * 128, k = k0 + (lane & 15) * 8;
    float m = 0.0f;
    if (k0 < K) {
        uint4 w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const uint4*>(src + ((int64_t)by * 16 + 4 * i + (lane >> 4)) * K + k);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t r = (int64_t)by * 16 + 4 * i + (lane >> 4);
            m = mag8(m, w[i]);
            *reinterpret_cast<uint2*>(s_q + r * K + k) = enc8(w[i], inv);
            uint32_t n0, n1;
            float a, b, d, e;
            select24_f32<SOFT>(w[i].x & 0xFFFFu, w[i].x >> 16, w[i].y & 0xFFFFu, w[i].y >> 16, n0, a, b);
            select24_f32<SOFT>(w[i].z & 0xFFFFu, w[i].z >> 16, w[i].w & 0xFFFFu, w[i].w >> 16, n1, d, e);
            const uint32_t q4 = fp8_enc2(a, b, inv) | (fp8_enc2(d, e, inv) << 16);
            uint32_t mw = n0 | (n1 << 4);                    // metadata of 32 k -> one store from every fourth lane
            mw |= row_shl<1>(mw) << 8;
            mw |= row_shl<2>(mw) << 16;
            if (codes) {
                *reinterpret_cast<uint32_t*>(codes + r * (K / 2) + k / 2) = q4;
                if ((lane & 3) == 0) *reinterpret_cast<uint32_t*>(meta + r * (K / 8) + k / 8) = mw;
            }
            *reinterpret_cast<uint32_t*>(codes_blk + blk_off(r, k / 4, K / 128)) = q4;      // 4 codes = 2 pairs
            if ((lane & 3) == 0) *reinterpret_cast<uint32_t*>(meta_blk + m8blk_off(r, k, K / 128)) = mw;
        }
    }
    note_part(amax, m, part);
}

// groups along the strided axis: S[r, k] = src[k * R + r]; 64 rows x 128 k through LDS, lane = (row, 32 k)
template <bool SOFT>
__device__ __forceinline__ void prune_cols_body(unsigned char* smem, int bx, int by, const uint16_t* __restrict__ src, int64_t R, int K, float inv, uint8_t* __restrict__ codes,
                                                uint8_t* __restrict__ meta, uint16_t* __restrict__ codes_blk, uint8_t* __restrict__ meta_blk, uint8_t* __restrict__ s_q,
                                                float* amax, float* part) {
    constexpr int P = kColsP;
    uint16_t* const tile = reinterpret_cast<uint16_t*>(smem);
    const int64_t r0 = (int64_t)bx * 64;
    const int k0 = by * 128, tid = threadIdx.x;
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int kk = tid / 8 + 32 * i, seg = tid % 8;
        const uint4 w = *reinterpret_cast<const uint4*>(src + (int64_t)(k0 + kk) * R + r0 + seg * 8);
        uint32_t* d = reinterpret_cast<uint32_t*>(&tile[kk * P + seg * 8]);
        d[0] = w.x; d[1] = w.y; d[2] = w.z; d[3] = w.w;
        m = mag8(m, w);
    }
    __syncthreads();
    const int rr = tid >> 2, q = tid & 3;
    uint32_t oc[4], mbytes = 0, sq[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        const uint16_t* p = &tile[(32 * q + 4 * g) * P + rr];
        uint32_t nib;
        float a, b;
        select24_f32<SOFT>(p[0], p[P], p[2 * P], p[3 * P], nib, a, b);
        sq[g] = fp8_enc2(bf2f(p[0]), bf2f(p[P]), inv) | (fp8_enc2(bf2f(p[2 * P]), bf2f(p[3 * P]), inv) << 16);
        const uint32_t c2 = fp8_enc2(a, b, inv);
        if (g & 1) oc[g >> 1] |= c2 << 16; else oc[g >> 1] = c2;
        mbytes |= nib << (4 * g);
    }
    const int64_t r = r0 + rr;
    const uint4 packed = make_uint4(oc[0], oc[1], oc[2], oc[3]);
    if (codes) {
        *reinterpret_cast<uint4*>(codes + r * (K / 2) + (k0 + 32 * q) / 2) = packed;
        *reinterpret_cast<uint32_t*>(meta + r * (K / 8) + (k0 + 32 * q) / 8) = mbytes;
    }
    *reinterpret_cast<uint4*>(codes_blk + blk_off(r, (k0 + 32 * q) / 4, K / 128)) = packed;       // 16 codes = 8 pairs
    *reinterpret_cast<uint32_t*>(meta_blk + m8blk_off(r, k0 + 32 * q, K / 128)) = mbytes;
    uint4* d = reinterpret_cast<uint4*>(s_q + r * K + k0 + 32 * q);
    d[0] = make_uint4(sq[0], sq[1], sq[2], sq[3]);
    d[1] = make_uint4(sq[4], sq[5], sq[6], sq[7]);
    note_part(amax, m, part);
}

}  // namespace

template <bool SOFT>
__global__ void __launch_bounds__(256) fp8_prologue_kernel(Fp8PrologueArgs a, int n_w2, int n_w1, int n_x) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kLds];
    __shared__ float part[4];
    int b = blockIdx.x;
    if (a.counters && b == 0) for (int k = threadIdx.x; k < kSplitCounters; k += 256) a.counters[k] = 0;
    if (b < n_w2) {
        const int gx = a.F / 64, per = gx * (a.D / 128), e = b / per, r = b - e * per;
        const int64_t o = (int64_t)e * a.F * a.D;
        prune_cols_body<SOFT>(smem, r % gx, r / gx, a.W2 + o, a.F, a.D, a.inv_w2, a.w2c ? a.w2c + o / 2 : nullptr, a.w2m ? a.w2m + o / 8 : nullptr,
                              reinterpret_cast<uint16_t*>(a.w2b + o / 2), a.w2mb + o / 8, a.w2q + o, a.amax_w2 ? a.amax_w2 + b : nullptr, part);
        return;
    }
    b -= n_w2;
    if (b < n_w1) {         // (a stack of experts is one tall matrix here: F is a multiple of 128)
        const int gx = (a.D + 511) / 512;
        prune_rows_body<SOFT>(b % gx, b / gx, a.W1, a.D, a.inv_w1, a.w1c, a.w1m, reinterpret_cast<uint16_t*>(a.w1b), a.w1mb, a.w1q, a.amax_w1 ? a.amax_w1 + b : nullptr, part);
        return;
    }
    b -= n_w1;
    const bool is_x = b < n_x;
    if (!is_x) b -= n_x;
    float* const slots = is_x ? a.slots_y2 : a.slots_dy1;
    if (b == 0 && slots && threadIdx.x < kAmaxSlots) slots[threadIdx.x * kAmaxSlotStride] = 0.0f;
    const int gx = a.D / 64;
    float* const am = is_x ? a.amax_x : a.amax_dy;
    quantize_body(smem, b % gx, b / gx, is_x ? a.X : a.dY, a.T, a.D, is_x ? a.inv_x : a.inv_dy, a.t_codes != 0, reinterpret_cast<uint16_t*>(is_x ? a.xt : a.dyt),
                  reinterpret_cast<uint16_t*>(is_x ? a.xq : a.dyq), am ? am + b : nullptr, part);
}

Fp8Parts fp8_parts(int64_t T, int64_t D, int64_t F, int64_t experts) {
    return {(int)(T / 64 * (D / 64)), (int)(experts * (F / 16) * ((D + 511) / 512)), (int)(experts * (F / 64) * (D / 128))};
}
hipError_t launch_fp8_prologue(const Fp8PrologueArgs& a, hipStream_t s) {
    if (a.T % 64 || a.D % 128 || a.F % 128) return hipErrorInvalidValue;
    const Fp8Parts n = fp8_parts(a.T, a.D, a.F, a.experts);
    const int n_w2 = a.W2 ? n.w2 : 0, n_w1 = a.W1 ? n.w1 : 0, n_x = a.X ? n.x : 0, all = n_w2 + n_w1 + n_x + (a.dY ? n.x : 0);
    if (all == 0) return hipSuccess;
    if (a.mode == 0) hipLaunchKernelGGL(fp8_prologue_kernel<false>, dim3((unsigned)all), dim3(256), 0, s, a, n_w2, n_w1, n_x);
    else             hipLaunchKernelGGL(fp8_prologue_kernel<true>, dim3((unsigned)all), dim3(256), 0, s, a, n_w2, n_w1, n_x);
    return hipGetLastError();
}

__global__ void __launch_bounds__(1024) amax_fold_kernel(AmaxFold a) {
    __shared__ unsigned char smem[64] __attribute__((aligned(16)));
    amax_fold_body<1024>(smem, blockIdx.x, a);
}
hipError_t launch_amax_fold(const AmaxFold& a, hipStream_t s) {
    hipLaunchKernelGGL(amax_fold_kernel, dim3((unsigned)a.count), dim3(1024), 0, s, a);
    return hipGetLastError();
}

}  // namespace sffn
