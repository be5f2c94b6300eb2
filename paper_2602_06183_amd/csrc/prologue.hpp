// The passes of a step that only depend on its inputs, as a unit (launch_mix.hpp): the transposed and blocked copies of X and dY (operands of eqs. (8), (1) and
// (5), (4)) and the pruning passes over W1 and W2.  HBM-bound at the large end; at the small one what counts is that they are few launches, or none of their own
// (forward_x.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"
#include "launch_mix.hpp"
#include "scans.hpp"

namespace sffn {

template <bool SOFT>
struct PrologueUnit {
    // workgroups of each part, the longest-running first (pruning of W2, of W1, then X and dY)
    struct Args { PrologueArgs a; int n_w2, n_w1, n_x, n_dy; };
    static constexpr int THREADS = 256, LDS = kPruneColsLds > kTransposeLds ? kPruneColsLds : kTransposeLds;
    static __device__ __forceinline__ void run(unsigned char* smem, int b, int, const Args& u) {
        const PrologueArgs& a = u.a;
        if (a.counters && b == 0) for (int k = threadIdx.x; k < kSplitCounters; k += 256) a.counters[k] = 0;
        if (b < u.n_w2) {         // 64 hidden units x 128 of d_model, matrix by matrix
            const int gx = a.F / 64, gy = (a.D + 127) / 128;
            const int e = b / (gx * gy), r = b - e * (gx * gy);
            prune24_cols_body<SOFT>(smem, r % gx, r / gx, e, a.W2, a.F, a.D, a.F, a.w2v, a.w2m, a.w2vb, a.w2mb, a.w2t);
            return;
        }
        b -= u.n_w2;
        if (b < u.n_w1) {         // 16 rows x 256 of d_model
            const int gx = (a.D / 64 + 3) / 4;
            prune24_rows_step_body<SOFT>(b % gx, b / gx, a.W1, a.D, a.D, a.w1v, a.w1m, a.w1vb, a.w1mb, 0, 0);
            return;
        }
        b -= u.n_w1;
        const int gx = a.D / 64;
        if (b < u.n_x) transpose_bf16_body(smem, b % gx, b / gx, a.X, a.T, a.D, a.D, a.xt, a.t_layout, a.xb, nullptr);
        else { b -= u.n_x; transpose_bf16_body(smem, b % gx, b / gx, a.dY, a.T, a.D, a.D, a.dyt, a.t_layout, a.dyb, nullptr); }
    }
    static Args make(const PrologueArgs& a) {
        const int n_t = (a.T / 64) * (a.D / 64);
        return {a, a.W2 ? a.experts * (a.F / 64) * ((a.D + 127) / 128) : 0, a.W1 ? a.experts * (a.F / 16) * ((a.D / 64 + 3) / 4) : 0, a.X ? n_t : 0, a.dY ? n_t : 0};
    }
    static unsigned count(const Args& u) { return (unsigned)(u.n_w2 + u.n_w1 + u.n_x + u.n_dy); }
    static const Args& args(const Args& u) { return u; }
};

}  // namespace sffn
