// Launchers of the pipelined tile kernel (gemm_v2_body.hpp) on bf16 operands in the blocked layout: eqs. (1), (4) with their V:N:M epilogues and
// the neuron-level router's grouped contractions.
#include "gemm_v2_body.hpp"

namespace sffn {

hipError_t launch_spmm_blocked(const uint16_t* a_vals, const uint8_t* a_meta, const uint16_t* B, const float* bias, int64_t Ra, int64_t Rb,
                               int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, bool past) {
    const GemmGroup g = grp ? *grp : GemmGroup();
    VnmEpilogue ep;
    ep.stream = past;
    if (out_i_contig || g.n > GemmGroup::kMaxExperts || (g.n && g.role == 2)) return hipErrorInvalidValue;
    return launch_gemm_v2<true, false, 0, true, false>({a_vals, a_meta, B, bias, (int)Ra, (int)Rb, (int)K, out, ldo, 0, 0, ep, g, 1.0f}, s);
}

// Dense operands, blocked: a load is 1 KB of consecutive bytes.  (Row-major ones were fetched as 64-byte halves of 16 lines: 8192 tokens, 4 experts, D = 2048, F = 8192
// 72 -> 60 us each for eqs. (5), (8).)
hipError_t launch_wgrad_router(const uint16_t* at, const uint16_t* G, int64_t Kc, int64_t N, int64_t rows, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup& grp) {
    if (!grp.n || grp.n > GemmGroup::kMaxExperts || grp.role != 2 || rows % 64 || Kc % 64 || N % 64) return hipErrorInvalidValue;
    return launch_gemm_v2<false, false, 0, true, false>({at, nullptr, G, nullptr, (int)Kc, (int)N, (int)rows, out, ldo, 0, 0, VnmEpilogue(), grp, 1.0f}, s);
}

hipError_t launch_gemm_vnm_epilogue(const uint16_t* a_vals, const uint8_t* a_meta, const uint16_t* B, const float* bias, int64_t F,
                                    int64_t T, int64_t K, uint16_t* out, const VnmEpilogue& ep, hipStream_t s, const GemmGroup* grp, int tile) {
    const GemmGroup g = grp ? *grp : GemmGroup();
    if (g.n && (g.n > GemmGroup::kMaxExperts || g.role != 1)) return hipErrorInvalidValue;
    if (ep.mode >= 5 && (ep.logM < 4 || ep.logM > 6)) return hipErrorInvalidValue;
    const GemmV2Args a = {a_vals, a_meta, B, bias, (int)F, (int)T, (int)K, out, F, 0, 0, ep, g, 1.0f};
#define SFFN_EPI(E) launch_gemm_v2<true, true, E, true, false>(a, s, tile)
    switch (ep.mode) {
        case 0: return SFFN_EPI(0);       // no V:N:M work: the dense output only
        case 1: return SFFN_EPI(1);
        case 2: return SFFN_EPI(2);
        case 3: return SFFN_EPI(3);
        case 4: return SFFN_EPI(4);
        // wide blocks: forward / backward epilogue for M = 16, 32, 64
        case 5: return ep.logM == 4 ? SFFN_EPI(20) : ep.logM == 5 ? SFFN_EPI(21) : SFFN_EPI(22);
        case 6: return ep.logM == 4 ? SFFN_EPI(36) : ep.logM == 5 ? SFFN_EPI(37) : SFFN_EPI(38);
        default: return hipErrorInvalidValue;
    }
#undef SFFN_EPI
}

}  // namespace sffn
