// Launchers of the V:2:8 activation GEMM (gemm_vnm8_body.hpp).
#include "gemm_vnm8_body.hpp"

namespace sffn {

bool vnm8_gemm_ok(int64_t T, int64_t N, int64_t F, int64_t ldw) {
    // (32-bit offsets inside the kernel: the dense operand and the offsets array stay below 2 GiB, so every offset is also a non-negative int)
    return T > 0 && T % 64 == 0 && N > 0 && N % 64 == 0 && F > 0 && F % 64 == 0 && ldw >= N && ldw % 8 == 0 && F * ldw * 2 < ((int64_t)1 << 31) &&
           T * F < ((int64_t)1 << 38);
}
bool vnm8_gemm_fp8_ok(int64_t T, int64_t N, int64_t F, int64_t ldw) {
    return T > 0 && T % 64 == 0 && N > 0 && N % 64 == 0 && F > 0 && F % 128 == 0 && ldw >= N && ldw % 16 == 0 && F * ldw < ((int64_t)1 << 31) &&
           T * F < ((int64_t)1 << 38);
}

// The large tile as 512 tokens x 128 columns or 256 x 256: the same work, 7 % faster in the first form (3 % on codes), which rounds segments of tokens up
// to more of them and columns to fewer; by the rounds of 256 workgroups that the call takes in either.  (8 experts of about 4100 tokens, D = 4096, F = 14336:
// 9 rounds in both, 1443 us and 1646.)
template <bool FP8>
static bool long_tile(const Vnm8Args& a) {
    const unsigned n256 = Vnm8Unit256<FP8>::count(a);
    return vnm8_rounds(Vnm8Unit512<FP8>::count(a), n256) < large_rounds(n256);
}

template <bool FP8>
static hipError_t launch_impl(Vnm8Args a, hipStream_t s, const GemmGroup* grp, int tile, const Split* split, bool past) {
    a.past = past;
    a.grp = grp ? *grp : GemmGroup();
    if (a.grp.n && (a.grp.role != 0 || a.grp.seg_dev || a.grp.n > GemmGroup::kMaxExperts)) return hipErrorInvalidValue;
    if (!tile) tile = pick_vnm8_tile(a.T, a.N, a.F / (FP8 ? 128 : 64), a.grp.n, FP8);
    if (split) a.split = *split;
    if (a.split.n > 1 && (a.grp.n || tile == 256)) return hipErrorInvalidValue;
    if (tile != 64 && a.split.n <= 1) {
        const AloneTiles& k = FP8 ? kAloneActivationFp8 : kAloneActivationBf16;
        const unsigned n512 = (unsigned)(0.93f * (float)Vnm8Unit512<FP8>::count(a)), n256 = Vnm8Unit256<FP8>::count(a);
        if (tall_alone(k, tile == 256 ? rounds_of_large(n512 < n256 ? n512 : n256, k.part) : 0.0f, Vnm8Unit128<FP8>::count(a), Vnm8UnitTall<FP8>::count(a), Vnm8UnitTall<FP8>::stages(a)))
            return launch_units<Vnm8UnitTall<FP8>>(s, a);
    }
    if (tile == 256) return long_tile<FP8>(a) ? launch_units<Vnm8Unit512<FP8>>(s, a) : launch_units<Vnm8Unit256<FP8>>(s, a);
    return tile == 128 ? launch_units<Vnm8Unit128<FP8>>(s, a) : launch_units<Vnm8Unit64<FP8>>(s, a);
}

hipError_t launch_vnm8_gemm(const uint16_t* vcb, const uint8_t* mcb, const uint8_t* cixt, const uint16_t* Wk, int64_t ldw, int64_t T, int64_t N,
                            int64_t F, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, int tile, const Split* split, bool past) {
    if (!vnm8_gemm_ok(T, N, F, ldw)) return hipErrorInvalidValue;
    return launch_impl<false>({vcb, mcb, cixt, reinterpret_cast<const uint8_t*>(Wk), (int)ldw, (int)T, (int)N, (int)F, out, ldo, 0, 0, GemmGroup(), 1.0f, Split()}, s, grp, tile, split, past);
}

hipError_t launch_vnm8_gemm_fp8(const uint8_t* vcb, const uint8_t* mcb, const uint8_t* cixt, const uint8_t* Wq, int64_t ldw, float alpha, int64_t T,
                                int64_t N, int64_t F, uint16_t* out, int64_t ldo, hipStream_t s, const GemmGroup* grp, int tile, const Split* split, bool past) {
    if (!vnm8_gemm_fp8_ok(T, N, F, ldw)) return hipErrorInvalidValue;
    return launch_impl<true>({reinterpret_cast<const uint16_t*>(vcb), mcb, cixt, Wq, (int)ldw, (int)T, (int)N, (int)F, out, ldo, 0, 0, GemmGroup(), alpha, Split()}, s, grp, tile, split, past);
}

}  // namespace sffn
