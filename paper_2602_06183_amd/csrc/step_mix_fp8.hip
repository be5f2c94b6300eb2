// Shared launches of the fp8 step with fp8 weight gradients and V:2:8 activations (StepTiles in kernels.hpp).
#include "step_mix.hpp"

namespace sffn {

hipError_t launch_step_mix_fp8_wide(int what, int logM, const StepTiles& t, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s, const AmaxFold* amax);

hipError_t launch_step_mix_fp8(int what, int logM, const StepTiles& t, const Vnm8Args* v8, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s,
                               const AmaxFold* amax) {
    if (logM != 3) return launch_step_mix_fp8_wide(what, logM, t, va, g, w, s, amax);
    using V = Units<Vnm8Unit64<true>, Vnm8Unit128<true>, Vnm8UnitTall<true>>;
    using W2 = Units<WgradUnit64<true, true, false>, WgradUnit128<true, true, false>, WgradUnitTall<true, true, false>>;
    using W1 = Units<WgradUnit64<true, false, false>, WgradUnit128<true, false, false>, WgradUnitTall<true, false, false>>;
    using G = Units<void, GemmV2Unit<true, true, 2, true, true, TileSel<true, 2>::T128>, GemmV2Unit<true, true, 2, true, true, TileTall>>;
    return launch_mix<true, true, V, W2, W1, G>(kMixFp8, what, t, v8, g, w, 64.0f, s, amax);
}

}  // namespace sffn
