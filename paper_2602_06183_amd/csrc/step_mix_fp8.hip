// Shared launches of the fp8 step with fp8 weight gradients (StepTiles in kernels.hpp).
#include "amax_fold.hpp"
#include "step_mix.hpp"

namespace sffn {

template <class V, int EPI, class W2, class W1, class VArgs>
static hipError_t pick(int what, const VArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s, const AmaxFold* amax) {
    using G = GemmV2Unit<true, true, EPI, true, true, typename TileSel<true, EPI>::T128>;
    if (what == kMixBackwardTail && amax) return launch_units<V, W1, AmaxUnit>(s, *v, w, *amax, wgrad_first<W1, V>(*v, w));
    return launch_mix<V, G, W2, W1>(what, v, g, w, s);
}
template <class V, int EPI, class VArgs>
static hipError_t pick_w(int what, const StepTiles& t, const VArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s, const AmaxFold* amax) {
    return t.w == 64 ? pick<V, EPI, WgradUnit64<true, true, false>, WgradUnit64<true, false, false>>(what, v, g, w, s, amax)
                     : pick<V, EPI, WgradUnit128<true, true, false>, WgradUnit128<true, false, false>>(what, v, g, w, s, amax);
}

hipError_t launch_step_mix_fp8(int what, int logM, const StepTiles& t, const Vnm8Args* v8, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s,
                               const AmaxFold* amax) {
    if (logM == 3) return t.v == 64 ? pick_w<Vnm8Unit64<true>, 2>(what, t, v8, g, w, s, amax) : pick_w<Vnm8Unit128<true>, 2>(what, t, v8, g, w, s, amax);
    return logM == 4 ? pick_w<GatherFp8Unit, 36>(what, t, va, g, w, s, amax) : logM == 5 ? pick_w<GatherFp8Unit, 37>(what, t, va, g, w, s, amax)
                                                                                  : pick_w<GatherFp8Unit, 38>(what, t, va, g, w, s, amax);
}

}  // namespace sffn
