// Launchers of the gathered-row activation GEMM (gemm_gather_body.hpp).
#include "gemm_gather_body.hpp"

namespace sffn {

bool vnm_spmm_gather_ok(int64_t T, int64_t N, int64_t F, int M) {
    const int64_t Kc = 4 * F / M;
    return M >= 8 && T % 64 == 0 && N % 64 == 0 && Kc % 64 == 0 && Kc <= kGMaxKc;
}

hipError_t launch_vnm_spmm_gather(const uint16_t* a_vals, const uint8_t* a_meta, const uint8_t* colidx, const uint16_t* Wk, int64_t ldw,
                                  int64_t T, int64_t N, int64_t F, int M, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, const Split* split, bool past) {
    if (!vnm_spmm_gather_ok(T, N, F, M) || ldw < N || F * ldw * 2 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    const GemmGroup g = grp ? *grp : GemmGroup();
    if (g.n && (g.role != 0 || g.seg_dev || g.n > GemmGroup::kMaxExperts)) return hipErrorInvalidValue;
    const int Kc = (int)(4 * F / M), logM = M == 8 ? 3 : M == 16 ? 4 : M == 32 ? 5 : 6;
    GatherArgs a = {a_vals, a_meta, colidx, Wk, (int)ldw, (int)T, (int)N, Kc, logM, 0, 1.0f, out, ldo, g, Split(), past};
    if (split) a.split = *split;
    if (a.split.n > 1 && (g.n || pick_gather_tile(T, N, Kc / 64) != 64)) return hipErrorInvalidValue;
    return pick_gather_tile(T, N, Kc / 64) == 64 ? launch_units<GatherUnit64>(s, a) : launch_units<GatherUnit256>(s, a);
}

bool vnm_spmm_gather_fp8_ok(int64_t T, int64_t N, int64_t F, int M) {
    const int64_t Kc = 4 * F / M;
    return M >= 8 && T % 64 == 0 && N % 64 == 0 && Kc % 128 == 0;
}

hipError_t launch_vnm_spmm_gather_fp8(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* colidx, const uint8_t* Wq, int64_t ldw, float alpha,
                                      int64_t T, int64_t N, int64_t F, int M, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, bool past) {
    if (!vnm_spmm_gather_fp8_ok(T, N, F, M) || ldw < N || ldw % 16 != 0 || F * ldw >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    const GemmGroup g = grp ? *grp : GemmGroup();
    if (g.n && (g.role != 0 || g.seg_dev || g.n > GemmGroup::kMaxExperts)) return hipErrorInvalidValue;
    const int Kc = (int)(4 * F / M), logM = M == 8 ? 3 : M == 16 ? 4 : M == 32 ? 5 : 6;
    return launch_units<GatherFp8Unit>(s, {a_codes, a_meta, colidx, Wq, (int)ldw, (int)T, (int)N, Kc, logM, 0, alpha, out, ldo, g, Split(), past});
}

}  // namespace sffn
