// Batches and tiles with spins as bits for the Philox kinds.
#include "ising_bits.h"

namespace rngx {

const void *batch_bits_kernel_philox(rngx_kind kind, uint32_t threads) {
    switch (kind) {
    case RNGX_PHILOX4X32_10: return batch_bits_kernel_of<PhiloxUnit>(threads);
    case RNGX_PHILOX4X32_7: return batch_bits_kernel_of<PhiloxUnit7>(threads);
    default: break;
    }
    return nullptr;
}

const void *tiles_kernel_philox(rngx_kind kind, bool hits) {
    switch (kind) {
    case RNGX_PHILOX4X32_10: return tiles_kernel_of<PhiloxUnit>(hits);
    case RNGX_PHILOX4X32_7: return tiles_kernel_of<PhiloxUnit7>(hits);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
