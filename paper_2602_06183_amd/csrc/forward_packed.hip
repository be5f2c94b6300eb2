// Eq. (1) of a forward call on packed weights and few tokens, X as it is: the launch that would copy X into blocks is left out, and what else that launch
// does (X.T for eq. (8) of a backward call that may follow, the counters of split contractions) rides along as workgroups of this one.
#include "gemm_v2_body.hpp"
#include "scans.hpp"

namespace sffn {

struct TransposeXUnit {
    using Args = TransposeX;
    static constexpr int THREADS = 256, LDS = kTransposeLds;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int, const Args& a) {
        if (a.counters && pid == 0) for (int k = threadIdx.x; k < kSplitCounters; k += 256) a.counters[k] = 0;
        const int gx = a.D / 64;
        transpose_bf16_body(smem, pid % gx, pid / gx, a.X, a.T, a.D, a.D, a.xt, a.t_layout, nullptr, nullptr);
    }
    static unsigned count(const Args& a) { return (unsigned)(a.T / 64 * (a.D / 64)); }
    static Args args(const Args& a) { return a; }
};

template <int EPI>
static hipError_t launch_impl(const GemmV2Args& a, const TransposeX& x, int tile, hipStream_t s) {
    using Sel = TileSel<true, EPI>;
    return tile == 64 ? launch_units<GemmV2Unit<true, true, EPI, true, false, typename Sel::T64, true>, TransposeXUnit>(s, a, x)
                      : launch_units<GemmV2Unit<true, true, EPI, true, false, typename Sel::T128, true>, TransposeXUnit>(s, a, x);
}

hipError_t launch_forward_packed(const uint16_t* a_vals, const uint8_t* a_meta, const float* bias, int64_t F, uint16_t* out, const VnmEpilogue& ep, const TransposeX& x,
                                 hipStream_t s, const GemmGroup* grp, int tile) {
    const GemmGroup g = grp ? *grp : GemmGroup();
    if (x.T % 64 || x.D % 64 || (tile != 64 && tile != 128) || (g.n && (g.n > GemmGroup::kMaxExperts || g.role != 1))) return hipErrorInvalidValue;
    const GemmV2Args a = {a_vals, a_meta, x.X, bias, (int)F, x.T, x.D, out, F, 0, 0, ep, g, 1.0f};
    if (ep.mode == 1) return launch_impl<1>(a, x, tile, s);
    if (ep.mode == 5 && ep.logM >= 4 && ep.logM <= 6) return ep.logM == 4 ? launch_impl<20>(a, x, tile, s) : ep.logM == 5 ? launch_impl<21>(a, x, tile, s) : launch_impl<22>(a, x, tile, s);
    return hipErrorInvalidValue;
}

}  // namespace sffn
