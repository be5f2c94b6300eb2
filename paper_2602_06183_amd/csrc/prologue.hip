// The step's preparing passes (prologue.hpp) in a launch of their own.  As four launches, each of which starts, fills and drains the chip, they took 17 us at
// T = 512, D = 256, F = 1024, where their bytes are worth 1 us.
#include "prologue.hpp"

namespace sffn {

hipError_t launch_step_prologue(const PrologueArgs& a, hipStream_t s) {
    if (a.T % 64 || a.D % 64 || a.F % 64) return hipErrorInvalidValue;
    return a.mode == 0 ? launch_units<PrologueUnit<false>>(s, PrologueUnit<false>::make(a)) : launch_units<PrologueUnit<true>>(s, PrologueUnit<true>::make(a));
}

}  // namespace sffn
