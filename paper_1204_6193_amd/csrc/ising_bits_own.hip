// Bit strips of the kinds with a map or multiplier of their own.
#include "ising_bits.h"

namespace rngx {

const void *bits_kernel_own(rngx_kind kind, int slots, bool hits, bool gang) {
    switch (kind) {
    case RNGX_LCG32_SUB: return bits_kernel_of<SmallUnit<Lcg32Sub>>(slots, hits, gang);
    case RNGX_LCG64_SUB: return bits_kernel_of<SmallUnit<Lcg64Sub>>(slots, hits, gang);
    case RNGX_MWC_DIFF: return bits_kernel_of<SmallUnit<MwcDiff>>(slots, hits, gang);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
