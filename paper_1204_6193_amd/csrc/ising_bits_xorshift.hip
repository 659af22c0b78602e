// Bit strips of XORWOW and XS1024W.
#include "ising_bits.h"

namespace rngx {

const void *bits_kernel_xorshift(rngx_kind kind, int slots, bool hits, bool gang) {
    switch (kind) {
    case RNGX_XORWOW: return bits_kernel_of<SmallUnit<Xorwow>>(slots, hits, gang);
    case RNGX_XS1024W: return bits_kernel_of<XsUnit>(slots, hits, gang);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
