// Bit strips of the Philox kinds.
#include "ising_bits.h"

namespace rngx {

const void *bits_kernel_philox(rngx_kind kind, int slots, bool hits, bool gang) {
    switch (kind) {
    case RNGX_PHILOX4X32_10: return bits_kernel_of<PhiloxUnit>(slots, hits, gang);
    case RNGX_PHILOX4X32_7: return bits_kernel_of<PhiloxUnit7>(slots, hits, gang);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
