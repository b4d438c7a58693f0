// Matrix product whose result is added straight into a permuted tensor (kernels in product.hip): host side.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "../../include/tperm.h"
#include "tperm_desc.h"

namespace tperm {

constexpr int kDepth = 16;    // summed indices per stage
// Workgroups per compute unit.  Smaller tiles and a third workgroup overlap the wait for memory of one
// with the arithmetic of another; 128 x 64 tiles of fp64 and two workgroups are 10 % faster on 4096^3 but
// 10 to 30 % slower where the destination has few columns.
constexpr int kResident = 3;

// One digit of a matrix index: the extent of the tensor dimension behind it and its stride (bytes)
// in the destination.
struct ProductDim {
    FastDiv div;
    uint32_t ext, stride;
};

// Descriptor of the kernel, passed by value.  "Fast" is the operand that holds the destination's
// stride-1 dimension: its index runs along the lanes of a wavefront.  Neighbouring lanes are neighbours
// in the destination where that dimension comes first in its operand's index, else they are not.
struct ProductDesc {
    uint32_t n_fast, n_slow, k;                  // extents of the product
    uint32_t splits, k_split;                    // the summed index in pieces of k_split
    uint32_t tiles_fast, tiles_slow, per_xcd;    // per_xcd: tiles one XCD takes
    uint32_t fast_bytes, slow_bytes, out_bytes;  // sizes of the three tensors
    uint32_t fast_dims, slow_dims;
    ProductDim fast[TPERM_DESC_MAX_DIMS], slow[TPERM_DESC_MAX_DIMS];
};

struct Product {
    ProductDesc d;
    int elem = 0;
    bool left_fast = true;                // the left operand is the fast one
    bool fast_k_first = false, slow_k_first = false;  // layout of the operands: summed index first?
    uint32_t run = 1;                     // neighbouring fast indices that lie side by side in the destination
    int vec = 1;                          // of those, how many one access moves: 1, 2, 4
    int shape = 0;                        // 0 wide tiles, 1 few fast indices, 2 few slow ones
    size_t tile_bytes = 0;
    size_t workspace = 0;                 // bytes for the partial products, if any
    bool pays = false;                    // expected to be faster than a library product and a transpose
};

// Nontemporal accesses to the destination: only for whole lines, and only where it does not fit the 256 MB
// memory-side cache with some room (78 MB of fp32, visited again after two others: 40 us cached, 47
// nontemporal).  Time against cached, destinations of 139 to 535 MB: 59 in runs of whole lines 0.93
// (0.81 to 1.02), 21 in longer runs of other lengths 1.16 (0.98 to 1.55).  Short runs lose most, since each
// piece of a line then goes to memory by itself: 253 MB in runs of 12 bytes 218 us cached, 1299 nontemporal.
constexpr uint32_t kCachedOutBytes = 128u << 20;
inline bool nontemporal_out(const Product& p, uintptr_t out) {
    return p.d.out_bytes > kCachedOutBytes && ((uint64_t)p.run * (uint64_t)p.elem | out) % 128u == 0;
}

// Host only: checks the arguments (as tperm_product_create) and fills the descriptor.
tperm_status_t build_product(Product* p, int rank, const int64_t* dims, const int* perm, int left_dims, int64_t k,
                             size_t elem, int left_k_first, int right_k_first);

}  // namespace tperm
