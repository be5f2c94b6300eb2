// Shared launches of the fp8 step with fp8 weight gradients and blocks of 16, 32, 64 columns (StepTiles in kernels.hpp).
#include "step_mix.hpp"

namespace sffn {

template <int EPI>
static hipError_t launch_impl(int what, const StepTiles& t, const GatherArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s, const AmaxFold* amax) {
    constexpr bool TALL = EPI == 38;              // M = 64: eq. (4) is on tall tiles as it is
    using V = Units<void, GatherFp8Unit, void>;
    using W2 = Units<WgradUnit64<true, true, false>, WgradUnit128<true, true, false>, WgradUnitTall<true, true, false>>;
    using W1 = Units<WgradUnit64<true, false, false>, WgradUnit128<true, false, false>, WgradUnitTall<true, false, false>>;
    using GT = GemmV2Unit<true, true, EPI, true, true, TileTall>;
    using G = std::conditional_t<TALL, Units<void, GT, void>, Units<void, GemmV2Unit<true, true, EPI, true, true, typename TileSel<true, EPI>::T128>, GT>>;
    MixTiles k = kMixWideFp8;
    if (TALL) k.g[0] = kMixTallFp8;
    return launch_mix<true, true, V, W2, W1, G>(k, what, t, v, g, w, 64.0f, s, amax);
}

hipError_t launch_step_mix_fp8_wide(int what, int logM, const StepTiles& t, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s, const AmaxFold* amax) {
    return logM == 4 ? launch_impl<36>(what, t, va, g, w, s, amax) : logM == 5 ? launch_impl<37>(what, t, va, g, w, s, amax) : launch_impl<38>(what, t, va, g, w, s, amax);
}

}  // namespace sffn
