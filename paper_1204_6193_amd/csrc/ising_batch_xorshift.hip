// Batches and tiles with spins as bits for XORWOW and XS1024W.
#include "ising_bits.h"

namespace rngx {

const void *batch_bits_kernel_xorshift(rngx_kind kind, uint32_t threads) {
    switch (kind) {
    case RNGX_XORWOW: return batch_bits_kernel_of<SmallUnit<Xorwow>>(threads);
    case RNGX_XS1024W: return batch_bits_kernel_of<XsUnit>(threads);
    default: break;
    }
    return nullptr;
}

const void *tiles_kernel_xorshift(rngx_kind kind, bool hits) {
    switch (kind) {
    case RNGX_XORWOW: return tiles_kernel_of<SmallUnit<Xorwow>>(hits);
    case RNGX_XS1024W: return tiles_kernel_of<XsUnit>(hits);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
