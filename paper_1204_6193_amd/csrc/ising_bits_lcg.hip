// Bit strips of the LCG and MWC kinds.
#include "ising_bits.h"

namespace rngx {

const void *bits_kernel_lcg(rngx_kind kind, int slots, bool hits, bool gang) {
    switch (kind) {
    case RNGX_LCG32: return bits_kernel_of<SmallUnit<Lcg32>>(slots, hits, gang);
    case RNGX_LCG64: return bits_kernel_of<SmallUnit<Lcg64>>(slots, hits, gang);
    case RNGX_MWC: return bits_kernel_of<SmallUnit<Mwc>>(slots, hits, gang);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
