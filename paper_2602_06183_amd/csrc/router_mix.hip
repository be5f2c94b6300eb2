// Shared launches of the router's step (where: router_shares() in kernels.hpp).  Its contractions are grouped by expert, so they have a few tiles more than fill the chip
// a whole number of times, and the last round of each is nearly empty: what does not depend on them fills it.
#include "gemm_v2_body.hpp"
#include "router_prologue.hpp"

namespace sffn {

using Plain = GemmV2Unit<true, false, 0, true, false, Tile<2, 2, 64, 3, 1>>;                        // eqs. (3), (7)
template <int EPI> using Epilogue = GemmV2Unit<true, true, EPI, true, false, Tile<2, 2, 64, 3, 1>>;      // eq. (1): 3, eq. (4): 4

struct TransposeUnit {
    struct Args { const uint16_t* in; int R, C; uint16_t* out; };
    static constexpr int THREADS = 256, LDS = kTransposeLds;
    static __device__ __forceinline__ void run(unsigned char* smem, int pid, int, const Args& a) {
        const int gx = a.C / 64;
        transpose_bf16_body(smem, pid % gx, pid / gx, a.in, a.R, a.C, a.C, a.out, 0, nullptr, nullptr);
    }
    static unsigned count(const Args& a) { return (unsigned)(a.R / 64 * (a.C / 64)); }
    static Args args(const Args& a) { return a; }
};

template <int LOGM>
static hipError_t launch_y1(const GemmV2Args& g1, const RouterPrologueArgs& p, hipStream_t s) {
    using Hard = RouterPrologueUnit<LOGM, false>;
    using Soft = RouterPrologueUnit<LOGM, true>;
    if (!Hard::fits(Hard::make(p))) return hipErrorInvalidValue;
    return p.mode == 0 ? launch_units<Epilogue<3>, Hard>(s, g1, Hard::make(p)) : launch_units<Epilogue<3>, Soft>(s, g1, Soft::make(p));
}
hipError_t launch_router_y1(const GemmV2Args& g1, const RouterPrologueArgs& p, hipStream_t s) {
    if (p.rows % 64 || p.D % 64 || p.F % (16 << p.logM)) return hipErrorInvalidValue;
    switch (p.logM) {
        case 3: return launch_y1<3>(g1, p, s);
        case 4: return launch_y1<4>(g1, p, s);
        case 5: return launch_y1<5>(g1, p, s);
        case 6: return launch_y1<6>(g1, p, s);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_router_dy2_y3(const GemmV2Args& g4, const GemmV2Args& g3, hipStream_t s) { return launch_units<Epilogue<4>, Plain>(s, g4, g3); }
hipError_t launch_router_dx(const GemmV2Args& g7, const uint16_t* dw2t, int64_t F, int64_t D, uint16_t* dW2, hipStream_t s) {
    if (F % 64 || D % 64) return hipErrorInvalidValue;
    return launch_units<Plain, TransposeUnit>(s, g7, {dw2t, (int)F, (int)D, dW2});
}

}  // namespace sffn
