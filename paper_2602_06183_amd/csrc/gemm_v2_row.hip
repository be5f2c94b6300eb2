// Launchers of the pipelined tile kernel (gemm_v2_body.hpp) on row-major operands: the stand-alone entry points.
#include "gemm_v2_body.hpp"

namespace sffn {

hipError_t launch_gemm_nt(int sparse_a, const uint16_t* a_vals, const uint8_t* a_meta, const uint16_t* B, const float* bias,
                             int64_t Ra, int64_t Rb, int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s) {
    const GemmV2Args a = {a_vals, a_meta, B, bias, (int)Ra, (int)Rb, (int)K, out, ldo, 0, 0, VnmEpilogue(), GemmGroup(), 1.0f};
    if (sparse_a) return out_i_contig ? launch_gemm_v2<true, true, 0, false, false>(a, s)
                                      : launch_gemm_v2<true, false, 0, false, false>(a, s);
    return out_i_contig ? launch_gemm_v2<false, true, 0, false, false>(a, s)
                        : launch_gemm_v2<false, false, 0, false, false>(a, s);
}

hipError_t launch_spmm24_fp8(const uint8_t* a_codes, const uint8_t* a_meta, const uint8_t* Bq, const float* bias, float alpha, int64_t Ra, int64_t Rb,
                             int64_t K, int out_i_contig, uint16_t* out, int64_t ldo, hipStream_t s) {
    if (K % 128 != 0) return hipErrorInvalidValue;
    // the kernel addresses its operands in 2-byte units: K / 2 of them per B row, K / 4 per A row
    const GemmV2Args a = {reinterpret_cast<const uint16_t*>(a_codes), a_meta, reinterpret_cast<const uint16_t*>(Bq), bias, (int)Ra, (int)Rb, (int)(K / 2), out, ldo,
                          0, 0, VnmEpilogue(), GemmGroup(), alpha};
    return out_i_contig ? launch_gemm_v2<true, true, 0, false, true>(a, s)
                        : launch_gemm_v2<true, false, 0, false, true>(a, s);
}

}  // namespace sffn
