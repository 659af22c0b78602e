// Batches and tiles with spins as bits for the LCG and MWC kinds.
#include "ising_bits.h"

namespace rngx {

const void *batch_bits_kernel_lcg(rngx_kind kind, uint32_t threads) {
    switch (kind) {
    case RNGX_LCG32: return batch_bits_kernel_of<SmallUnit<Lcg32>>(threads);
    case RNGX_LCG64: return batch_bits_kernel_of<SmallUnit<Lcg64>>(threads);
    case RNGX_MWC: return batch_bits_kernel_of<SmallUnit<Mwc>>(threads);
    default: break;
    }
    return nullptr;
}

const void *tiles_kernel_lcg(rngx_kind kind, bool hits) {
    switch (kind) {
    case RNGX_LCG32: return tiles_kernel_of<SmallUnit<Lcg32>>(hits);
    case RNGX_LCG64: return tiles_kernel_of<SmallUnit<Lcg64>>(hits);
    case RNGX_MWC: return tiles_kernel_of<SmallUnit<Mwc>>(hits);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
