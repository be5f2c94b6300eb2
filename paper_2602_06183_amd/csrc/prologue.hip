// The passes of a step that only depend on its inputs, as one launch: the transposed and blocked copies of X and dY (operands of eqs. (8), (1) and
// (5), (4)) and the pruning passes over W1 and W2.  Separately they are four launches that each start, fill and drain the chip: 17 us at
// T = 512, D = 256, F = 1024, where their bytes are worth 1 us.  HBM-bound at the large end.
#include "common.hpp"
#include "kernels.hpp"
#include "scans.hpp"

namespace sffn {

// n_w2, n_w1, n_x: workgroups of each part, the longest-running first (pruning of W2, of W1, then X and dY)
template <bool SOFT>
__global__ void __launch_bounds__(256) step_prologue_kernel(PrologueArgs a, int n_w2, int n_w1, int n_x) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[kPruneColsLds > kTransposeLds ? kPruneColsLds : kTransposeLds];
    int b = blockIdx.x;
    if (a.counters && b == 0) for (int k = threadIdx.x; k < kSplitCounters; k += 256) a.counters[k] = 0;
    if (b < n_w2) {         // 64 hidden units x 128 of d_model, matrix by matrix
        const int gx = a.F / 64, gy = (a.D + 127) / 128;
        const int e = b / (gx * gy), r = b - e * (gx * gy);
        prune24_cols_body<SOFT>(smem, r % gx, r / gx, e, a.W2, a.F, a.D, a.F, a.w2v, a.w2m, a.w2vb, a.w2mb, a.w2t);
        return;
    }
    b -= n_w2;
    if (b < n_w1) {         // 16 rows x 256 of d_model
        const int gx = (a.D / 64 + 3) / 4;
        prune24_rows_step_body<SOFT>(b % gx, b / gx, a.W1, a.D, a.D, a.w1v, a.w1m, a.w1vb, a.w1mb, 0, 0);
        return;
    }
    b -= n_w1;
    const int gx = a.D / 64;
    if (b < n_x) transpose_bf16_body(smem, b % gx, b / gx, a.X, a.T, a.D, a.D, a.xt, a.t_layout, a.xb, nullptr);
    else { b -= n_x; transpose_bf16_body(smem, b % gx, b / gx, a.dY, a.T, a.D, a.D, a.dyt, a.t_layout, a.dyb, nullptr); }
}

hipError_t launch_step_prologue(const PrologueArgs& a, hipStream_t s) {
    if (a.T % 64 || a.D % 64 || a.F % 64) return hipErrorInvalidValue;
    const int n_t = (a.T / 64) * (a.D / 64);
    const int n_w2 = a.W2 ? a.experts * (a.F / 64) * ((a.D + 127) / 128) : 0, n_w1 = a.W1 ? a.experts * (a.F / 16) * ((a.D / 64 + 3) / 4) : 0;
    const int n_x = a.X ? n_t : 0, n = n_w2 + n_w1 + n_x + (a.dY ? n_t : 0);
    if (n == 0) return hipSuccess;
    if (a.mode == 0) hipLaunchKernelGGL((step_prologue_kernel<false>), dim3((unsigned)n), dim3(256), 0, s, a, n_w2, n_w1, n_x);
    else             hipLaunchKernelGGL((step_prologue_kernel<true>), dim3((unsigned)n), dim3(256), 0, s, a, n_w2, n_w1, n_x);
    return hipGetLastError();
}

}  // namespace sffn
