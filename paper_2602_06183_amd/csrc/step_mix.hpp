// Which units share a launch: see StepTiles in kernels.hpp.
#pragma once
#include <type_traits>
#include "amax_fold.hpp"
#include "gemm_gather_body.hpp"
#include "gemm_v2_body.hpp"
#include "gemm_vnm8_body.hpp"
#include "gemm_wgrad_body.hpp"

namespace sffn {

// Eqs. (5), (8) before eqs. (3), (7) where their tiles are the longer ones: begun behind a round of the others they end the launch alone.  A tile's length is the stages that one
// wavefront contracts (T = 3072, D = 448, F = 1792, M = 16: 48 of eq. (5), 2 of eq. (3), one workgroup a CU: 48 us with eq. (3) first, 25 with eq. (5) first).
template <class W, class V, class VArgs>
bool wgrad_first(const VArgs& v, const WgradArgs& w) { return W::stages(w) > V::stages(v); }

// A contraction's units: its 64 tile, its 128 tile and its tall one (void: not built)
template <class U64_, class U128_, class Tall_> struct Units { using U64 = U64_; using U128 = U128_; using Tall = Tall_; };
template <class T> struct Tag { using type = T; };
template <class U> constexpr bool kBuilt = !__is_same(U, void);
template <class U, class F>
hipError_t with_unit(bool on64, bool tall, F f) {
    if constexpr (kBuilt<typename U::U64>) if (on64) return f(Tag<typename U::U64>());
    if constexpr (kBuilt<typename U::Tall>) if (tall) return f(Tag<typename U::Tall>());
    return f(Tag<typename U::U128>());
}
template <class U, class Args>
MixCount mix_count(bool on64, const Args& a) {
    if constexpr (kBuilt<typename U::U64>) if (on64) return {U::U64::count(a), 0, 0, U::U64::stages(a)};
    unsigned tall = 0;
    if constexpr (kBuilt<typename U::Tall>) tall = U::Tall::count(a);
    return {0, U::U128::count(a), tall, U::U128::stages(a)};
}

// V, W2, W1, G: the units of eqs. (3) / (7), (5) (out_i_contig), (8), (4); FORWARD: whole steps too; k: their times; slots: workgroups at a time on an XCD; AMAX: amax may say that
// the last launch folds the step's maxima
template <bool FORWARD, bool AMAX, class V, class W2, class W1, class G, class VArgs>
hipError_t launch_mix(const MixTiles& k, int what, const StepTiles& t, const VArgs* v, const GemmV2Args* g, const WgradArgs& w, float slots, hipStream_t s, const AmaxFold* amax = nullptr) {
    const bool v64 = t.v == 64, w64 = t.w == 64;
    const float bytes = 2.0f * ((float)w.F * (float)w.N * (what == kMixBackwardTail ? 2.0f : 3.6f) + (float)w.T * (2.0f * (float)w.N + (float)w.F));
    const unsigned form = mix_form(k, what, what != kMixBackwardHead ? mix_count<V>(v64, *v) : MixCount(), mix_count<W2>(w64, w), what != kMixBackwardTail ? mix_count<G>(false, *g) : MixCount(), slots, bytes);
    const bool v_tall = form & 1, w_tall = form & 2, g_tall = form & 4;
    if (what == kMixBackwardTail)
        return with_unit<V>(v64, v_tall, [&](auto tv) {
            return with_unit<W1>(w64, w_tall, [&](auto tw) {
                using VU = typename decltype(tv)::type; using WU = typename decltype(tw)::type;
                if constexpr (AMAX) if (amax) return launch_units<VU, WU, AmaxUnit>(s, *v, w, *amax, wgrad_first<WU, VU>(*v, w));
                return launch_units<VU, WU>(s, *v, w, wgrad_first<WU, VU>(*v, w));
            });
        });
    if (what == kMixBackwardHead) {
        if constexpr (kBuilt<typename G::Tall>) if (g_tall) return launch_units<typename W2::Tall, typename G::Tall>(s, w, *g);
        return with_unit<W2>(w64, w_tall, [&](auto tw) { return launch_units<typename decltype(tw)::type, typename G::U128>(s, w, *g); });
    }
    if constexpr (FORWARD) if (what == kMixForwardTail) {
        if constexpr (kBuilt<typename G::Tall>) if (g_tall) {        // (eqs. (5) and, where it has them, (3) on tall tiles too)
            using VU = std::conditional_t<kBuilt<typename V::Tall>, typename V::Tall, typename V::U128>; using WU = typename W2::Tall;
            return launch_units<VU, WU, typename G::Tall>(s, *v, w, *g, wgrad_first<WU, VU>(*v, w));
        }
        return with_unit<V>(v64, v_tall, [&](auto tv) {
            return with_unit<W2>(w64, w_tall, [&](auto tw) {
                using VU = typename decltype(tv)::type; using WU = typename decltype(tw)::type;
                return launch_units<VU, WU, typename G::U128>(s, *v, w, *g, wgrad_first<WU, VU>(*v, w));
            });
        });
    }
    return hipErrorInvalidValue;
}

}  // namespace sffn
