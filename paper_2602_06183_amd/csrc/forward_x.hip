// Eq. (1) on X as it is, and in the same launch the preparing passes that only later launches read (X.T, dY, W2, the counters of split contractions): a launch
// in front of eq. (1) is left for the pruning of W1 only, and not even that on packed weights or (behind.W1) where eq. (1) prunes what it reads itself.
#include "gemm_v2_body.hpp"
#include "prologue.hpp"

namespace sffn {

template <int EPI, bool SOFT>
static hipError_t launch_impl(const GemmV2Args& a, const PrologueArgs& behind, int tile, hipStream_t s) {
    using Sel = TileSel<true, EPI>;
    using P = PrologueUnit<SOFT>;
    if constexpr (EPI == 1)
        if (behind.W1) {
            GemmV2Args raw = a;
            raw.a_vals = behind.W1;
            raw.grp.a_stride = (int64_t)behind.F * behind.D;
            return behind.D <= 256 ? launch_units<GemmV2Unit<true, true, EPI, true, false, Tile<1, 1, 64, 1, 4>, true, false, SOFT ? 2 : 1>, P>(s, raw, P::make(behind))
                                   : launch_units<GemmV2Unit<true, true, EPI, true, false, Tile<1, 1, 64, 2, 4>, true, false, SOFT ? 2 : 1>, P>(s, raw, P::make(behind));
        }
    return tile == 64 ? launch_units<GemmV2Unit<true, true, EPI, true, false, typename Sel::T64, true>, P>(s, a, P::make(behind))
                      : launch_units<GemmV2Unit<true, true, EPI, true, false, typename Sel::T128, true>, P>(s, a, P::make(behind));
}
template <int EPI>
static hipError_t launch_mode(const GemmV2Args& a, const PrologueArgs& behind, int tile, hipStream_t s) {
    return behind.mode == 0 ? launch_impl<EPI, false>(a, behind, tile, s) : launch_impl<EPI, true>(a, behind, tile, s);
}

hipError_t launch_forward_x(const uint16_t* a_vals, const uint8_t* a_meta, const float* bias, const uint16_t* X, uint16_t* out, const VnmEpilogue& ep,
                            const PrologueArgs& behind, hipStream_t s, const GemmGroup* grp, int tile) {
    const GemmGroup g = grp ? *grp : GemmGroup();
    const PrologueArgs& p = behind;
    if (p.T % 64 || p.D % 64 || p.F % 64 || (tile != 64 && tile != 128) || (p.W1 && (tile != 64 || p.D > 512 || ep.mode != 1)) || (g.n && (g.n > GemmGroup::kMaxExperts || g.role != 1))) return hipErrorInvalidValue;
    const GemmV2Args a = {a_vals, a_meta, X, bias, p.F, p.T, p.D, out, p.F, 0, 0, ep, g, 1.0f};
    if (ep.mode == 1) return launch_mode<1>(a, p, tile, s);
    if (ep.mode == 5 && ep.logM >= 4 && ep.logM <= 6) return ep.logM == 4 ? launch_mode<20>(a, p, tile, s) : ep.logM == 5 ? launch_mode<21>(a, p, tile, s) : launch_mode<22>(a, p, tile, s);
    return hipErrorInvalidValue;
}

}  // namespace sffn
