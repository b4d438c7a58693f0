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
// stride-1 dimension: its index runs along the lanes of a wavefront.
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
    int vec = 1;                          // destination elements that lie side by side: 1, 2, 4
    int shape = 0;                        // 0 wide tiles, 1 few fast indices, 2 few slow ones
    size_t tile_bytes = 0;
    size_t workspace = 0;                 // bytes for the partial products, if any
    bool pays = false;                    // expected to be faster than a library product and a transpose
};

// Host only: checks the arguments (as tperm_product_create) and fills the descriptor.
tperm_status_t build_product(Product* p, int rank, const int64_t* dims, const int* perm, int left_dims, int64_t k,
                             size_t elem, int left_k_first, int right_k_first);

}  // namespace tperm
