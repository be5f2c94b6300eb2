// Which units share a launch: see StepTiles in kernels.hpp.
#pragma once
#include "gemm_gather_body.hpp"
#include "gemm_v2_body.hpp"
#include "gemm_vnm8_body.hpp"
#include "gemm_wgrad_body.hpp"

namespace sffn {

// V, G, W2, W1: the units of eqs. (3) / (7), (4), (5) (out_i_contig) and (8)
template <class V, class G, class W2, class W1, class VArgs>
hipError_t launch_mix(int what, const VArgs* v, const GemmV2Args* g, const WgradArgs& w, hipStream_t s) {
    switch (what) {
        case kMixForwardTail: return launch_units<V, W2, G>(s, *v, w, *g);
        case kMixBackwardHead: return launch_units<W2, G>(s, w, *g);
        case kMixBackwardTail: return launch_units<V, W1>(s, *v, w);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sffn
