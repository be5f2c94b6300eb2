// Shared launches of the bf16 step with V:2:8 activations (StepTiles in kernels.hpp).
#include "step_mix.hpp"

namespace sffn {

hipError_t launch_step_mix_bf16_wide(int what, int logM, const StepTiles& t, bool acc32, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s);

template <bool ACC32>
static hipError_t launch_impl(int what, const StepTiles& t, const Vnm8Args* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    using V = Units<Vnm8Unit64<false>, Vnm8Unit128<false>, Vnm8UnitTall<false>>;
    using W2 = Units<WgradUnit64<false, true, ACC32>, WgradUnit128<false, true, ACC32>, WgradUnitTall<false, true, ACC32>>;
    using W1 = Units<WgradUnit64<false, false, ACC32>, WgradUnit128<false, false, ACC32>, WgradUnitTall<false, false, ACC32>>;
    using G = Units<void, GemmV2Unit<true, true, 2, true, false, TileSel<true, 2>::T128>, GemmV2Unit<true, true, 2, true, false, TileTall>>;
    // (64 tiles of eqs. (5), (8): 156,672 bytes of LDS, one workgroup a CU)
    MixTiles k = ACC32 ? kMixBf16Sums : kMixBf16;
    if (w.grp.n) k.few = 0.0f;
    return launch_mix<!ACC32, false, V, W2, W1, G>(k, what, t, v, g, w, t.w == 64 ? 32.0f : 64.0f, s);
}

hipError_t launch_step_mix_bf16(int what, int logM, const StepTiles& t, bool acc32, const Vnm8Args* v8, const GatherArgs* va, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    if (logM != 3) return launch_step_mix_bf16_wide(what, logM, t, acc32, va, g, w, s);
    return acc32 ? launch_impl<true>(what, t, v8, g, w, s) : launch_impl<false>(what, t, v8, g, w, s);
}

}  // namespace sffn
