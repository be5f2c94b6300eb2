// Launchers of the pipelined tile kernel (gemm_v2_body.hpp) on fp8 codes in the blocked layout: eqs. (1), (4) of the fp8 step.
#include "gemm_v2_body.hpp"

namespace sffn {

hipError_t launch_gemm_fp8_blocked(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* Bq, const float* bias, float alpha, int64_t Ra,
                                   int64_t Rb, int64_t K, uint16_t* out, int64_t ldo, const VnmEpilogue* ep, hipStream_t s, const GemmGroup* grp, int tile) {
    if (K % 128 != 0 || !ep) return hipErrorInvalidValue;
    if (ep->mode >= 5 && (ep->logM < 4 || ep->logM > 6)) return hipErrorInvalidValue;
    const GemmGroup g = grp ? *grp : GemmGroup();
    // grouped: the tokens are the j rows (role 1: A = the expert's packed weights)
    if (g.n && (g.n > GemmGroup::kMaxExperts || g.role != 1 || g.seg_dev)) return hipErrorInvalidValue;
    const GemmV2Args a = {reinterpret_cast<const uint16_t*>(a_codes), a_meta, reinterpret_cast<const uint16_t*>(Bq), bias, (int)Ra, (int)Rb, (int)(K / 2), out, ldo,
                          0, 0, *ep, g, alpha};
#define SFFN_F8(E) launch_gemm_v2<true, true, E, true, true>(a, s, tile)
    switch (ep->mode) {
        case 1: return SFFN_F8(1);
        case 2: return SFFN_F8(2);
        case 5: return ep->logM == 4 ? SFFN_F8(20) : ep->logM == 5 ? SFFN_F8(21) : SFFN_F8(22);
        case 6: return ep->logM == 4 ? SFFN_F8(36) : ep->logM == 5 ? SFFN_F8(37) : SFFN_F8(38);
        default: return hipErrorInvalidValue;
    }
#undef SFFN_F8
}

}  // namespace sffn
