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
    // Up to 256 summed indices the one kernel wins (334 of 700 seeded contractions: 1.9 to 2.3 times the
    // speed up to 128, 1.3 to 1.5 up to 256, the slowest 0.87); beyond that it is taken where the
    // estimates say so: one of the other 366 is slower then, by 13 %, the rest 1.5 times as fast together
    // (always taken, 55 would be slower, by up to 28 %).
    p->pays = d.k <= 256 || best <= library_us(d, p->elem);
    return TPERM_OK;
}

}  // namespace tperm
