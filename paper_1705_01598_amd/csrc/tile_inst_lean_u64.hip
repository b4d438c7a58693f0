// Instantiations of the tile kernel's lean form (see NO_MASKS there) for uint64_t elements: plain
// LDS-staged tiles of 256 threads, 6 to 16 slots per thread, the four cache policies.
#include "tile_kernel.hpp"

namespace tperm {

template <int NREG>
static const void* lean_kernel_ptr(int nt) {
    typedef uint64_t T;
    switch (nt) {
        case 0: return reinterpret_cast<const void*>(&tile_kernel<T, NREG, 256, true, 0, false, false, false, false, false, true>);
        case 1: return reinterpret_cast<const void*>(&tile_kernel<T, NREG, 256, true, 1, false, false, false, false, false, true>);
        case 2: return reinterpret_cast<const void*>(&tile_kernel<T, NREG, 256, true, 2, false, false, false, false, false, true>);
        default: return reinterpret_cast<const void*>(&tile_kernel<T, NREG, 256, true, 3, false, false, false, false, false, true>);
    }
}

const void* tile_kernel_lean_u64(int nreg, int nt) {
    switch (nreg) {
        case 6: return lean_kernel_ptr<6>(nt);
        case 7: return lean_kernel_ptr<7>(nt);
        case 8: return lean_kernel_ptr<8>(nt);
        case 10: return lean_kernel_ptr<10>(nt);
        case 12: return lean_kernel_ptr<12>(nt);
        case 14: return lean_kernel_ptr<14>(nt);
        case 16: return lean_kernel_ptr<16>(nt);
        default: return nullptr;
    }
}

}  // namespace tperm
