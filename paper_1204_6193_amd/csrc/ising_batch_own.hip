// Batches and tiles with spins as bits for the kinds with a map or multiplier of their own.
#include "ising_bits.h"

namespace rngx {

const void *batch_bits_kernel_own(rngx_kind kind, uint32_t threads) {
    switch (kind) {
    case RNGX_LCG32_SUB: return batch_bits_kernel_of<SmallUnit<Lcg32Sub>>(threads);
    case RNGX_LCG64_SUB: return batch_bits_kernel_of<SmallUnit<Lcg64Sub>>(threads);
    case RNGX_MWC_DIFF: return batch_bits_kernel_of<SmallUnit<MwcDiff>>(threads);
    default: break;
    }
    return nullptr;
}

const void *tiles_kernel_own(rngx_kind kind, bool hits) {
    switch (kind) {
    case RNGX_LCG32_SUB: return tiles_kernel_of<SmallUnit<Lcg32Sub>>(hits);
    case RNGX_LCG64_SUB: return tiles_kernel_of<SmallUnit<Lcg64Sub>>(hits);
    default: break;
    }
    return nullptr;
}

}  // namespace rngx
