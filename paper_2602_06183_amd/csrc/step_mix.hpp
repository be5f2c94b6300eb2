// Which units share a launch: see StepTiles in kernels.hpp.
#pragma once
#include "gemm_gather_body.hpp"
#include "gemm_v2_body.hpp"
#include "gemm_vnm8_body.hpp"
#include "gemm_wgrad_body.hpp"

namespace sffn {

// Eqs. (5), (8) before eqs. (3), (7) where their tiles are the longer ones: begun behind a round of the others they end the launch alone.  A tile's length is the stages that one
// wavefront contracts (T = 3072, D = 448, F = 1792, M = 16: 48 of eq. (5), 2 of eq. (3), one workgroup a CU: 48 us with eq. (3) first, 25 with eq. (5) first).
template <class W, class V, class VArgs>
bool wgrad_first(const VArgs& v, const WgradArgs& w) { return W::stages(w) > V::stages(v); }

// V, G, W2, W1: the units of eqs. (3) / (7), (4), (5) (out_i_contig) and (8)
template <class V, class G, class W2, class W1, class VArgs>
hipError_t launch_mix(int what, const VArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    switch (what) {
        case kMixForwardTail: return launch_units<V, W2, G>(s, *v, w, *g, wgrad_first<W2, V>(*v, w));
        case kMixBackwardHead: return launch_units<W2, G>(s, w, *g);
        case kMixBackwardTail: return launch_units<V, W1>(s, *v, w, wgrad_first<W1, V>(*v, w));
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sffn
