// The end of the fp8 step's amax collection: out[i] = the largest of n[i] floats, stride[i] apart (a preparing pass's one value per workgroup, an
// epilogue's slots; n = 0: 0).  One workgroup per tensor; in shapes whose contractions share launches it rides in the last of them.
#pragma once
#include "kernels.hpp"

namespace sffn {

template <int NT>
__device__ __forceinline__ void amax_fold_body(unsigned char* smem, int i, const AmaxFold& a) {
    float* const part = reinterpret_cast<float*>(smem);
    const float* p = a.p[i];
    const int n = a.n[i], stride = a.stride[i];
    float m = 0.0f;
#pragma unroll 8
    for (int k = threadIdx.x; k < n; k += NT) m = __builtin_fmaxf(m, p[(int64_t)k * stride]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NT / 64; ++w) m = __builtin_fmaxf(m, part[w]);
        a.out[i] = m;
    }
}
struct AmaxUnit {
    using Args = AmaxFold;
    static constexpr int THREADS = 256, LDS = 64;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int, const Args& a) { amax_fold_body<THREADS>(smem, pid, a); }
    static unsigned count(const Args& a) { return (unsigned)a.count; }
    static Args args(const Args& a) { return a; }
};

}  // namespace sffn
