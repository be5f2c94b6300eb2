// Shared launches of the bf16 step with blocks of 16, 32, 64 columns (StepTiles in kernels.hpp).
#include "step_mix.hpp"

namespace sffn {

template <class V, bool ACC32, int EPI>
static hipError_t pick(int what, const GatherArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    using G = GemmV2Unit<true, true, EPI, true, false, typename TileSel<true, EPI>::T128>;
    using W2 = WgradUnit128<false, true, ACC32>;
    using W1 = WgradUnit128<false, false, ACC32>;
    if constexpr (ACC32) if (what == kMixForwardTail) return hipErrorInvalidValue;
    if (what == kMixBackwardTail) return launch_units<V, W1>(s, *v, w, wgrad_first<W1, V>(*v, w));
    if constexpr (ACC32) return launch_units<W2, G>(s, w, *g);
    else return launch_mix<V, G, W2, W1>(what, v, g, w, s);
}
template <class V, bool ACC32>
static hipError_t pick_m(int what, int logM, const GatherArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    return logM == 4 ? pick<V, ACC32, 36>(what, v, g, w, s) : logM == 5 ? pick<V, ACC32, 37>(what, v, g, w, s) : pick<V, ACC32, 38>(what, v, g, w, s);
}

hipError_t launch_step_mix_bf16_wide(int what, int logM, const StepTiles& t, bool acc32, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    if (t.v == 64) return acc32 ? pick_m<GatherUnit64, true>(what, logM, va, g, w, s) : pick_m<GatherUnit64, false>(what, logM, va, g, w, s);
    return acc32 ? pick_m<GatherUnit256, true>(what, logM, va, g, w, s) : pick_m<GatherUnit256, false>(what, logM, va, g, w, s);
}

}  // namespace sffn
