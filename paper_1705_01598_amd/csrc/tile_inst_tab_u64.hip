// Instantiations of the tile kernel with positions from tables (see TAB there) for uint64_t elements.
#include "tile_kernel.hpp"

namespace tperm {

const void* tile_kernel_tab_u64(int nreg, int nt, bool acc, bool vec2, bool lean) {
    return tile_kernel_tab_select<uint64_t>(nreg, nt, acc, vec2, lean);
}

}  // namespace tperm
