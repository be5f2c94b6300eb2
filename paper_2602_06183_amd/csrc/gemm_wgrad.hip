// Launchers of the weight-gradient contractions (gemm_wgrad_body.hpp).
#include "gemm_wgrad_body.hpp"

namespace sffn {

template <bool FP8, bool OUT_I_CONTIG, bool ACC32>
static hipError_t launch_sized(const WgradArgs& a, hipStream_t s, int tile) {
    if constexpr (!FP8) if (wgrad_three_a_cu(a.F, a.N, a.T, a.grp.n, tile)) return launch_units<WgradUnit<FP8, OUT_I_CONTIG, ACC32, WTile<2, 2, 64, 2, 1>>>(s, a);
    if constexpr (!FP8) {
        using Tall = WgradUnitTall<false, OUT_I_CONTIG, ACC32>;
        const unsigned n256 = WgradUnit256<false, OUT_I_CONTIG, ACC32>::count(a);
        if (tile != 64 && tall_alone(kAloneGradientBf16, tile == 256 ? rounds_of_large(n256, kAloneGradientBf16.part) : 0.0f, WgradUnit128<false, OUT_I_CONTIG, ACC32>::count(a), Tall::count(a), Tall::stages(a)))
            return launch_units<Tall>(s, a);
    }
    if (tile == 256) return launch_units<WgradUnit256<FP8, OUT_I_CONTIG, ACC32>>(s, a);
    if (tile == 128) return launch_units<WgradUnit128<FP8, OUT_I_CONTIG, ACC32>>(s, a);
    return launch_units<WgradUnit64<FP8, OUT_I_CONTIG, ACC32>>(s, a);
}
template <bool FP8>
static hipError_t launch_impl(WgradArgs a, int out_i_contig, hipStream_t s, const GemmGroup* grp, bool acc32, bool split_ok, int tile) {
    a.grp = grp ? *grp : GemmGroup();
    if (a.T % 64 != 0 || a.T <= 0 || (a.grp.n && (a.grp.n > GemmGroup::kMaxExperts || a.grp.role != 2))) return hipErrorInvalidValue;
    if (!tile) tile = pick_wgrad_tile(a.F, a.N, a.T, a.grp.n, split_ok, FP8);
    if (out_i_contig) return acc32 ? launch_sized<FP8, true, true>(a, s, tile) : launch_sized<FP8, true, false>(a, s, tile);
    return acc32 ? launch_sized<FP8, false, true>(a, s, tile) : launch_sized<FP8, false, false>(a, s, tile);
}

hipError_t launch_wgrad_vnm_fp8(const uint8_t* atc, const uint8_t* kmask, const uint8_t* Gq, float alpha, int64_t F, int64_t N, int64_t T,
                                int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, bool acc32, bool split_ok, int tile) {
    return launch_impl<true>({reinterpret_cast<const uint16_t*>(atc), kmask, reinterpret_cast<const uint16_t*>(Gq), alpha, (int)F, (int)N, (int)T, out, ldo, 0, 0, GemmGroup()},
                             out_i_contig, s, grp, acc32, split_ok, tile);
}

hipError_t launch_wgrad_vnm(const uint16_t* atc, const uint8_t* kmask, const uint16_t* G, int64_t F, int64_t N, int64_t T,
                            int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, bool acc32, bool split_ok, int tile) {
    return launch_impl<false>({atc, kmask, G, 1.0f, (int)F, (int)N, (int)T, out, ldo, 0, 0, GemmGroup()}, out_i_contig, s, grp, acc32, split_ok, tile);
}

}  // namespace sffn
