// Shared launches of the bf16 step with V:2:8 activations (StepTiles in kernels.hpp).
#include "step_mix.hpp"

namespace sffn {

hipError_t launch_step_mix_bf16_wide(int what, int logM, const StepTiles& t, bool acc32, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s);

template <class V, bool ACC32, class W2, class W1>
static hipError_t pick(int what, const Vnm8Args* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    using G = GemmV2Unit<true, true, 2, true, false, TileSel<true, 2>::T128>;
    if constexpr (ACC32) if (what == kMixForwardTail) return hipErrorInvalidValue;
    if constexpr (ACC32) return what == kMixBackwardHead ? launch_units<W2, G>(s, w, *g) : launch_units<V, W1>(s, *v, w, wgrad_first<W1, V>(*v, w));
    else return launch_mix<V, G, W2, W1>(what, v, g, w, s);
}
template <class V, bool ACC32>
static hipError_t pick_w(int what, const StepTiles& t, const Vnm8Args* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    return t.w == 64 ? pick<V, ACC32, WgradUnit64<false, true, ACC32>, WgradUnit64<false, false, ACC32>>(what, v, g, w, s)
                     : pick<V, ACC32, WgradUnit128<false, true, ACC32>, WgradUnit128<false, false, ACC32>>(what, v, g, w, s);
}

hipError_t launch_step_mix_bf16(int what, int logM, const StepTiles& t, bool acc32, const Vnm8Args* v8, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    if (logM != 3) return launch_step_mix_bf16_wide(what, logM, t, acc32, va, g, w, s);
    if (t.v == 64) return acc32 ? pick_w<Vnm8Unit64<false>, true>(what, t, v8, g, w, s) : pick_w<Vnm8Unit64<false>, false>(what, t, v8, g, w, s);
    return acc32 ? pick_w<Vnm8Unit128<false>, true>(what, t, v8, g, w, s) : pick_w<Vnm8Unit128<false>, false>(what, t, v8, g, w, s);
}

}  // namespace sffn
