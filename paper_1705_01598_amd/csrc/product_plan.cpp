// Plan of a matrix product that is added into a permuted tensor (kernels in product.hip): index digits,
// tile shape, pieces of the summed index, and whether it pays.  Host code only, without HIP.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "plan.hpp"
#include "product.hpp"

namespace tperm {

constexpr int kComputeUnits = 256;
// Most pieces of the summed index, and most tiles times pieces (48 MB of partial products).
constexpr uint32_t kMaxPieces = 96;
constexpr uint64_t kMaxUnits = 1536;

// Estimated microseconds: rounds of resident workgroups, each a chain of stages that takes at least the
// round trip of its panels and, once the matrix cores are shared, its share of them; then the sum of
// the partial products.  Fitted to 1192 timings of 300 seeded contractions with 1 to 96 pieces (mean
// error 13 %); the number of pieces that it picks is 3 % (fp32) and 7 % (fp64) off the best one.
static double product_us(int elem, double units, uint32_t depth, bool split) {
    const double share = std::min((double)kResident, units / kComputeUnits);
    const double stage = elem == 8 ? std::max(1.03, 0.606 * share) : std::max(1.22, 0.229 * share);
    const double rounds = std::ceil(units / (kComputeUnits * kResident));
    const double sum = elem == 8 ? 4.7 + 0.0054 * units : 1.9 + 0.019 * units;
    return (elem == 8 ? 5.0 : 1.9) + rounds * depth / kDepth * stage + (split ? sum : 0.0);
}

// The same for the library's product and the transpose that adds it: its rate on large products, a
// floor for small ones, where the host is the bound (fp64 products also run along the summed index), two
// passes over the product.
static double library_us(const ProductDesc& d, int elem) {
    const double flops = 2.0 * d.n_fast * d.n_slow * (double)d.k;
    const double gemm = elem == 8 ? std::max({18.0, flops / 58e6, 0.035 * d.k}) : std::max(20.0, flops / 140e6);
    return gemm + 2.0 * d.out_bytes / 4.5e6;
}

// A split product of wide fp64 tiles, closer than product_us: a stage costs what the fullest compute unit
// takes for it, and the pieces are summed from memory.  95 seeded products: standard deviation 8 %.
static double split_f64_us(double units, uint32_t depth) {
    const double share = std::min((double)kResident, std::ceil(units / kComputeUnits));
    const double rounds = std::ceil(units / (kComputeUnits * kResident));
    return 3.3 + rounds * ((depth + kDepth - 1) / kDepth) * std::max(1.03, 0.69 * share) + 2.5 + 0.0147 * units;
}

// Whether the dimensions of one index are listed in the destination's order.
static bool in_order(const ProductDim* dim, uint32_t n) {
    for (uint32_t z = 1; z < n; ++z)
        if (dim[z].stride < dim[z - 1].stride) return false;
    return true;
}

// Whether the one kernel is expected to be faster than the library's product and an accumulating transpose
// (us: its estimate).  Times are of the library's way / of the one kernel.
//  - Not where the destination's stride-1 dimension is not the first of its operand: each lane then
//    reaches a line of its own (121 seeded products: 24 slower, by up to 6 times).
//  - Not in short runs of a larger destination where an operand's dimensions are listed in another order than
//    the destination's: the pieces of a line come from different tiles (30 seeded products: 8 slower, by up to 3.8
//    times; in order, 55 such: 1.14 at the least).
//  - Not where fp64 products of few tiles fill the library's tiles: of seven slower contractions in 1270, six were
//    fp64 in two to four pieces with both extents above 250 (0.82 to 0.90); they leave by the estimate above.
//  - Else up to 256 summed indices, and beyond where the estimates say so.
// 1450 seeded contractions with new seeds (extents of the workload families, any extents, plain matrices, first
// extents of 2 to 8): 841 with K <= 128 2.19, all taken, 0.99 at the least; 106 of 107 up to 256 1.68, three below 0.97,
// 0.89 at the least; beyond, 287 taken 2.46, 0.99 at the least, 215 not taken, of which 77 would be slower.
constexpr uint32_t kAnyOrderRunBytes = 64, kAnyOrderOutBytes = 8u << 20, kLibraryTiles = 150;
static bool one_kernel_pays(const Product& p, double us) {
    const ProductDesc& d = p.d;
    if (d.fast_dims > 0 && d.fast[0].stride != (uint32_t)p.elem) return false;
    if (p.run * (uint32_t)p.elem < kAnyOrderRunBytes && d.out_bytes > kAnyOrderOutBytes &&
        !(in_order(d.fast, d.fast_dims) && in_order(d.slow, d.slow_dims)))
        return false;
    const double library = library_us(d, p.elem);
    if (p.elem == 8 && d.splits > 1 && std::min(d.n_fast, d.n_slow) >= kLibraryTiles &&
        split_f64_us((double)d.tiles_fast * d.tiles_slow * d.splits, d.k_split) > 0.9 * library)
        return false;
    return d.k <= 256 || us <= library;
}

// Tile shape: wide tiles, or one of the thin ones where an index has so few values that wide tiles are
// mostly padding.  Thin tiles read more per result, so their padded area counts double and more.  Over
// 700 seeded contractions (time of the pick / best of the three, geometric mean): wide tiles always
// 1.12, this rule 1.02.
static void choose_shape(Product* p) {
    ProductDesc& d = p->d;
    const uint32_t tile[3][2] = {{128, p->elem == 8 ? 32u : 64u}, {16, p->elem == 8 ? 128u : 256u}, {256, 16}};
    const double weight[3] = {1.0, d.k >= 256 ? 2.0 : 3.0, 2.5};
    double least = 0.0;
    for (int i = 0; i < (p->elem == 8 ? 2 : 3); ++i) {
        const uint32_t nf = (d.n_fast + tile[i][0] - 1u) / tile[i][0], ns = (d.n_slow + tile[i][1] - 1u) / tile[i][1];
        const double area = weight[i] * nf * tile[i][0] * ((double)ns * tile[i][1]);
        if (i == 0 || area < least) {
            least = area;
            p->shape = i;
            d.tiles_fast = nf;
            d.tiles_slow = ns;
            p->tile_bytes = (size_t)tile[i][0] * tile[i][1] * (size_t)p->elem;
        }
    }
}

tperm_status_t build_product(Product* p, int rank, const int64_t* dims, const int* perm, int left_dims, int64_t k,
                             size_t elem, int left_k_first, int right_k_first) {
    tperm_status_t st = validate(rank, dims, perm, elem);
    if (st != TPERM_OK) return st;
    if (left_dims < 0 || left_dims > rank) return TPERM_ERR_RANK;
    if (k < 1) return TPERM_ERR_DIMS;
    int64_t ext[2] = {1, 1};  // of the left and right index
    for (int z = 0; z < rank; ++z) ext[z < left_dims ? 0 : 1] *= dims[z];
    const int64_t limit = (((int64_t)1 << 32) - 256) / (int64_t)elem;
    if (ext[0] * ext[1] >= limit || k >= limit || ext[0] * k >= limit || ext[1] * k >= limit) return TPERM_ERR_TOO_LARGE;
    // the digits of either index, in the order of the index, with their strides in the destination
    int64_t stride[TPERM_MAX_RANK], s = (int64_t)elem;
    for (int j = 0; j < rank; ++j) {
        stride[perm[j]] = s;
        s *= dims[perm[j]];
    }
    std::memset(&p->d, 0, sizeof(p->d));
    ProductDim digits[2][TPERM_MAX_RANK];
    uint32_t n_digits[2] = {0, 0};
    for (int z = 0; z < rank; ++z) {
        if (dims[z] == 1) continue;
        const int side = z < left_dims ? 0 : 1;
        uint32_t& n = n_digits[side];
        ProductDim* last = n > 0 ? &digits[side][n - 1] : nullptr;
        if (last != nullptr && stride[z] == (int64_t)last->stride * last->ext) {
            last->ext *= (uint32_t)dims[z];  // travels with the digit in front of it
            last->div = make_fastdiv(last->ext);
        } else {
            digits[side][n++] = ProductDim{make_fastdiv((uint32_t)dims[z]), (uint32_t)dims[z], (uint32_t)stride[z]};
        }
    }
    // fast side: the one that holds the destination's stride-1 dimension, at whatever place
    p->left_fast = true;
    for (int j = 0; j < rank; ++j)
        if (dims[perm[j]] > 1) {
            p->left_fast = perm[j] < left_dims;
            break;
        }
    const int fast = p->left_fast ? 0 : 1, slow = 1 - fast;
    ProductDesc& d = p->d;
    p->elem = (int)elem;
    p->fast_k_first = (p->left_fast ? left_k_first : right_k_first) != 0;
    p->slow_k_first = (p->left_fast ? right_k_first : left_k_first) != 0;
    d.n_fast = (uint32_t)ext[fast];
    d.n_slow = (uint32_t)ext[slow];
    d.k = (uint32_t)k;
    d.fast_dims = n_digits[fast];
    d.slow_dims = n_digits[slow];
    std::memcpy(d.fast, digits[fast], sizeof(ProductDim) * n_digits[fast]);
    std::memcpy(d.slow, digits[slow], sizeof(ProductDim) * n_digits[slow]);
    d.fast_bytes = (uint32_t)(ext[fast] * k * (int64_t)elem);
    d.slow_bytes = (uint32_t)(ext[slow] * k * (int64_t)elem);
    d.out_bytes = (uint32_t)(ext[0] * ext[1] * (int64_t)elem);
    p->run = d.fast_dims > 0 && d.fast[0].stride == (uint32_t)elem ? d.fast[0].ext : 1u;
    p->vec = p->run % 4 == 0 && elem == 4 ? 4 : (p->run % 2 == 0 ? 2 : 1);
    choose_shape(p);
    if (p->shape == 1) p->vec = 1;  // a lane holds one element of a row there
    const uint64_t tiles = (uint64_t)d.tiles_fast * d.tiles_slow;
    // the summed index in pieces where the tiles alone leave compute units idle
    double best = 0.0;
    for (uint32_t n = 1; n == 1 || (n <= kMaxPieces && tiles * n <= kMaxUnits && d.k / n >= 2u * kDepth); ++n) {
        const uint32_t depth = n == 1 ? d.k : ((d.k + n - 1u) / n + kDepth - 1u) / kDepth * kDepth;
        const uint32_t pieces = (d.k + depth - 1u) / depth;
        const double us = product_us(p->elem, (double)tiles * pieces, depth, pieces > 1u);
        if (n == 1 || us < best) {
            best = us;
            d.splits = pieces;
            d.k_split = depth;
        }
    }
    p->workspace = d.splits > 1u ? (size_t)tiles * d.splits * p->tile_bytes : 0;
    d.per_xcd = (uint32_t)((tiles * d.splits + 7u) / 8u);
    p->pays = one_kernel_pays(*p, best);
    return TPERM_OK;
}

}  // namespace tperm
