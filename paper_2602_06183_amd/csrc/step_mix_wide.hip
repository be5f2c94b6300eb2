// Shared launches of the bf16 step with blocks of 16, 32, 64 columns (StepTiles in kernels.hpp).
#include "step_mix.hpp"

namespace sffn {

template <bool ACC32, int EPI>
static hipError_t launch_impl(int what, const StepTiles& t, const GatherArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    constexpr bool TALL = EPI == 38;              // M = 64: eq. (4) is on tall tiles as it is
    using V = Units<GatherUnit64, GatherUnit256, void>;
    using W2 = Units<void, WgradUnit128<false, true, ACC32>, WgradUnitTall<false, true, ACC32>>;
    using W1 = Units<void, WgradUnit128<false, false, ACC32>, WgradUnitTall<false, false, ACC32>>;
    using GT = GemmV2Unit<true, true, EPI, true, false, TileTall>;
    using G = std::conditional_t<TALL, Units<void, GT, void>, Units<void, GemmV2Unit<true, true, EPI, true, false, typename TileSel<true, EPI>::T128>, GT>>;
    MixTiles k = ACC32 ? kMixWideBf16Sums : kMixWideBf16;
    if (TALL) k.g[0] = kMixTallBf16;
    return launch_mix<!ACC32, false, V, W2, W1, G>(k, what, t, v, g, w, 64.0f, s);
}
template <bool ACC32>
static hipError_t launch_m(int what, int logM, const StepTiles& t, const GatherArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    return logM == 4 ? launch_impl<ACC32, 36>(what, t, v, g, w, s) : logM == 5 ? launch_impl<ACC32, 37>(what, t, v, g, w, s) : launch_impl<ACC32, 38>(what, t, v, g, w, s);
}

hipError_t launch_step_mix_bf16_wide(int what, int logM, const StepTiles& t, bool acc32, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    return acc32 ? launch_m<true>(what, logM, t, va, g, w, s) : launch_m<false>(what, logM, t, va, g, w, s);
}

}  // namespace sffn
