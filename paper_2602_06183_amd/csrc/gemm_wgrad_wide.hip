// Launchers of the weight-gradient contractions for blocks of M = 32, 64 columns (gemm_wgrad_wide_body.hpp).
#include "gemm_wgrad_wide_body.hpp"

namespace sffn {

// 512 x 64 tiles; 512 x 32 (two workgroups per CU) where the larger ones do not fill the chip
template <bool OUT_I_CONTIG, bool ACC32, int LOGM>
static hipError_t launch_m(const WgradArgs& a, hipStream_t s) {
    using Large = WgradWideUnit<OUT_I_CONTIG, ACC32, WideTile<LOGM, 512, 64, LOGM == 5 ? 2 : 1, LOGM == 5 ? 6 : 4>>;
    using Small = WgradWideUnit<OUT_I_CONTIG, ACC32, WideTile<LOGM, 512, 32, 1, 4>>;
    return Large::count(a) >= 256 ? launch_units<Large>(s, a) : launch_units<Small>(s, a);
}
template <bool OUT_I_CONTIG, bool ACC32>
static hipError_t launch_sized(const WgradArgs& a, int logM, hipStream_t s) {
    return logM == 5 ? launch_m<OUT_I_CONTIG, ACC32, 5>(a, s) : launch_m<OUT_I_CONTIG, ACC32, 6>(a, s);
}

hipError_t launch_wgrad_wide(const uint16_t* at_kept, const uint8_t* colidx, const uint16_t* G, int64_t F, int64_t N, int64_t T, int logM, int out_i_contig, uint16_t* out,
                             int64_t ldo, hipStream_t s, const GemmGroup* grp, bool acc32) {
    const WgradArgs a = {at_kept, colidx, G, 1.0f, (int)F, (int)N, (int)T, out, ldo, 0, 0, grp ? *grp : GemmGroup()};
    if (T % 64 != 0 || T <= 0 || N % 64 != 0 || logM < 5 || logM > 6 || (4 * F >> logM) % 32 != 0) return hipErrorInvalidValue;
    if (a.grp.n && (a.grp.n > GemmGroup::kMaxExperts || a.grp.role != 2)) return hipErrorInvalidValue;
    if (out_i_contig) return acc32 ? launch_sized<true, true>(a, logM, s) : launch_sized<true, false>(a, logM, s);
    return acc32 ? launch_sized<false, true>(a, logM, s) : launch_sized<false, false>(a, logM, s);
}

}  // namespace sffn
