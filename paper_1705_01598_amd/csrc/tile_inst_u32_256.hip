// Instantiations of the tile kernel for uint32_t elements, 256-thread workgroups.
#include "tile_kernel.hpp"

namespace tperm {

const void* tile_kernel_u32_256(int nreg, bool use_lds, int nt, bool align, bool acc, bool loads_first, bool vec2, bool steady) {
    if (steady) return tile_kernel_select<uint32_t, 256, true>(nreg, use_lds, nt, align, acc, loads_first, vec2);
    return tile_kernel_select<uint32_t, 256>(nreg, use_lds, nt, align, acc, loads_first, vec2);
}

}  // namespace tperm
