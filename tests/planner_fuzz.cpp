// Host-only fuzz driver for the planners, meant to be built with AddressSanitizer and
// UndefinedBehaviorSanitizer (see test_planner_host.py).  It links plan.cpp, model.cpp and
// product_plan.cpp alone (none has a HIP dependency), creates plans for random problems and options,
// and checks every plan's index map for being a bijection of 0..vol-1, and every product's offsets
// against the permutation.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "../paper_1705_01598_amd/csrc/plan.hpp"
#include "../paper_1705_01598_amd/csrc/product.hpp"

// Byte offset of index i of one side, as the kernels compute it.
static uint64_t digits_offset(const tperm::ProductDim* dim, uint32_t n, uint32_t i) {
    uint64_t at = 0;
    for (uint32_t z = 0; z < n; ++z) {
        const uint32_t quot = tperm::fdiv(i, dim[z].div);
        at += (uint64_t)(i - quot * dim[z].ext) * dim[z].stride;
        i = quot;
    }
    return at;
}

// Plans of products: 0 = all right, else the iteration that is wrong.
static int fuzz_products(int iters, int* made, int* rejected) {
    std::mt19937_64 rng(54321);
    for (int it = 1; it <= iters; ++it) {
        const bool big = it % 8 == 0;  // up to and beyond the limits; only the ends of each index are checked
        const int rank = 1 + (int)(rng() % (it % 5 == 0 ? 16 : 6));
        int64_t dims[TPERM_MAX_RANK];
        int perm[TPERM_MAX_RANK];
        int64_t vol = 1;
        const int64_t most = big ? (int64_t)1 << 31 : 1 << 16;
        for (int z = 0; z < rank; ++z) {
            dims[z] = 1 + (int64_t)(rng() % (big ? 4000 : (rank > 6 ? 4 : 40)));
            if (vol * dims[z] > most) dims[z] = 1;
            vol *= dims[z];
            perm[z] = z;
        }
        for (int z = rank - 1; z > 0; --z) std::swap(perm[z], perm[rng() % (z + 1)]);
        const int left = (int)(rng() % (rank + 1));
        const size_t elem = rng() % 2 ? 4 : 8;
        const int64_t k = it % 97 == 0 ? INT64_MAX >> (rng() % 40) : (int64_t)1 << (rng() % (big ? 31 : 14)) | (int64_t)(rng() % 64);
        int64_t ext[2] = {1, 1};
        for (int z = 0; z < rank; ++z) ext[z < left ? 0 : 1] *= dims[z];
        tperm::Product p;
        const tperm_status_t st = tperm::build_product(&p, rank, dims, perm, left, k, elem, (int)(rng() % 2), (int)(rng() % 2));
        const int64_t limit = (((int64_t)1 << 32) - 256) / (int64_t)elem;
        const bool fits = vol < limit && k < limit && ext[0] * k < limit && ext[1] * k < limit;
        if (st != (fits ? TPERM_OK : TPERM_ERR_TOO_LARGE)) return it;
        if (!fits) {
            ++*rejected;
            continue;
        }
        const tperm::ProductDesc& d = p.d;
        const int fast = p.left_fast ? 0 : 1;
        if (d.n_fast != (uint64_t)ext[fast] || d.n_slow != (uint64_t)ext[1 - fast] || d.k != (uint64_t)k) return it;
        // the pieces start at whole stages, none is empty, together they are the summed index
        if (d.splits < 1 || (uint64_t)(d.splits - 1) * d.k_split >= d.k || (uint64_t)d.splits * d.k_split < d.k ||
            (d.splits > 1 && d.k_split % tperm::kDepth != 0))
            return it;
        const uint64_t tiles = (uint64_t)d.tiles_fast * d.tiles_slow;
        const uint32_t tile_f = p.shape == 1 ? 16 : (p.shape == 2 ? 256 : 128);
        const uint32_t tile_s = (uint32_t)(p.tile_bytes / elem / tile_f);
        if (d.tiles_fast != (d.n_fast + tile_f - 1) / tile_f || d.tiles_slow != (d.n_slow + tile_s - 1) / tile_s) return it;
        if ((uint64_t)d.per_xcd * 8 < tiles * d.splits || tiles * d.splits + 8 > UINT32_MAX) return it;
        if (p.workspace != (d.splits > 1 ? tiles * d.splits * p.tile_bytes : 0)) return it;
        int owner = 0;  // of the destination's stride-1 dimension
        for (int j = rank - 1; j >= 0; --j)
            if (dims[perm[j]] > 1) owner = perm[j] < left ? 0 : 1;
        if (fast != owner) return it;
        // offsets, against strides computed one dimension at a time
        uint64_t stride[TPERM_MAX_RANK], s = elem;
        for (int j = 0; j < rank; ++j) {
            stride[perm[j]] = s;
            s *= (uint64_t)dims[perm[j]];
        }
        for (int side = 0; side < 2; ++side) {
            const int of = side == 0 ? fast : 1 - fast;
            const uint32_t n = (uint32_t)ext[of], step = big ? std::max(1u, n / 1000) : 1u;
            const tperm::ProductDim* dim = side == 0 ? d.fast : d.slow;
            const uint32_t n_dims = side == 0 ? d.fast_dims : d.slow_dims;
            for (uint32_t i = 0; i < n; i = i + step < n || i == n - 1 ? i + step : n - 1) {
                uint64_t want = 0, rem = i;
                for (int z = of == 0 ? 0 : left; z < (of == 0 ? left : rank); ++z) {
                    want += rem % (uint64_t)dims[z] * stride[z];
                    rem /= (uint64_t)dims[z];
                }
                if (digits_offset(dim, n_dims, i) != want || want >= d.out_bytes) return it;
                // neighbours that one access moves lie side by side
                if (side == 0 && p.vec > 1 && i % (uint32_t)p.vec != 0 && step == 1 &&
                    digits_offset(dim, n_dims, i - 1) + elem != want)
                    return it;
            }
            if (side == 0 && n % (uint32_t)p.vec != 0) return it;
        }
        // nontemporal accesses to whole lines of a large destination only
        bool lines = d.out_bytes > tperm::kCachedOutBytes;
        for (uint32_t i = 0; lines && i < std::min(d.n_fast, 4096u); ++i)
            lines = i % (128u / (uint32_t)elem) == 0 ? digits_offset(d.fast, d.fast_dims, i) % 128 == 0
                                                     : digits_offset(d.fast, d.fast_dims, i - 1) + elem == digits_offset(d.fast, d.fast_dims, i);
        for (uint32_t i = 0; lines && i < std::min(d.n_slow, 4096u); ++i) lines = digits_offset(d.slow, d.slow_dims, i) % 128 == 0;
        if (tperm::nontemporal_out(p, 4096) && !lines) return it;
        if (tperm::nontemporal_out(p, 4096 + 64)) return it;
        ++*made;
    }
    return 0;
}

int main(int argc, char** argv) {
    const int iters = argc > 1 ? atoi(argv[1]) : 400;
    std::mt19937_64 rng(12345);
    int made = 0, rejected = 0, windows = 0, pair_windows = 0, images = 0;
    for (int it = 0; it < iters; ++it) {
        const int rank = 1 + (int)(rng() % 16);
        int64_t dims[TPERM_MAX_RANK];
        int perm[TPERM_MAX_RANK];
        int64_t vol = 1;
        for (int z = 0; z < rank; ++z) {
            const int64_t cap = rank > 8 ? 3 : (rank > 4 ? 7 : 40);
            dims[z] = 1 + (int64_t)(rng() % cap);
            if (vol * dims[z] > 200000) dims[z] = 1;
            vol *= dims[z];
            perm[z] = z;
        }
        for (int z = rank - 1; z > 0; --z) std::swap(perm[z], perm[rng() % (z + 1)]);
        // every fourth problem of rank 2-4 gets a long leading output dim, so that the
        // line-aligned window form (chunks of whole lines along it) can apply
        const bool long_q0 = rank >= 2 && rank <= 4 && (it % 4) == 3 && perm[0] != 0;
        if (long_q0) {
            vol /= dims[perm[0]];
            dims[perm[0]] = 40 + (int64_t)(rng() % 300);
            for (int z = 0; z < rank && vol * dims[perm[0]] > 400000; ++z)
                if (z != perm[0] && dims[z] > 1) {
                    vol /= dims[z];
                    dims[z] = 1 + dims[z] / 4;
                    vol *= dims[z];
                }
            vol *= dims[perm[0]];
        }
        tperm_plan_opts_t o;
        std::memset(&o, 0, sizeof(o));
        o.lds_pad = -1;
        const size_t elem = ((it / 4) & 1) ? 4 : 8;
        const int mode = long_q0 ? 2 : (int)(rng() % 4);
        if (mode == 1) o.kernel_class = 1 + (int)(rng() % 5);
        if (mode == 0 && (rng() % 2)) o.selector = 1;  // tile chosen by the analytical model
        if (mode >= 2) {
            o.kernel_class = TPERM_KERNEL_PACKED;
            o.m = 1 + (int)(rng() % rank);
            o.k = 1 + (int)(rng() % rank);
            o.tile_in = (int64_t)(rng() % 50);
            o.tile_out = (int64_t)(rng() % 50);
            o.grid_mode = (int)(rng() % 9);
            o.window_in = (int)(rng() % 20);
            o.window_out = (int)(rng() % 20);
            o.threads = (rng() % 2) ? 64 : 256;
            o.lds_buffers = (int)(rng() % 3);
            o.align_out = (int)(rng() % 3);
            if (long_q0) {
                o.align_out = 2;
                // make the line-aligned window form likely: one leading output dim in the
                // tile, chunked in whole 128-byte lines
                o.k = 1;
                o.tile_out = (int64_t)(128 / (int)elem) * (1 + (int64_t)(rng() % 3));
                if (rng() % 2) o.tile_in &= ~(int64_t)1;  // pairs need an even tile extent
                o.threads = 256;
                o.vec2 = 0;
            }
            o.lds_pad = (int)(rng() % 8) - 1;
            o.vec2 = (int)(rng() % 3);
            if (long_q0 && elem == 4 && (rng() % 2)) {
                // pairs inside the windows: one input dim in the tile, even extent along it
                o.vec2 = 2;
                o.m = 1;
                o.tile_in = 2 + 2 * (int64_t)(rng() % 24);
            }
            o.loads_first = (int)(rng() % 3);
            o.tile_order = (int)(rng() % 3);
        }
        if ((rng() % 5) == 0) o.large = 1;  // planned the way tensors of 4 GiB and more are
        tperm::Plan* p = nullptr;
        const tperm_status_t st = tperm::create_plan(&p, rank, dims, perm, elem, &o);
        if (st != TPERM_OK) {
            if (st != TPERM_ERR_KERNEL) {
                std::printf("unexpected status %d at iteration %d\n", (int)st, it);
                return 1;
            }
            ++rejected;
            continue;
        }
        if (o.large == 1 && p->kclass != TPERM_KERNEL_COPY &&
            (!p->big || p->loads_first || (p->kclass != TPERM_KERNEL_NAIVE && (!p->use_lds || p->threads != 256)))) {
            std::printf("a large plan uses a form large tensors have no kernel for, iteration %d\n", it);
            return 1;
        }
        std::vector<int64_t> map((size_t)vol);
        const tperm_status_t ms = tperm::index_map(*p, map.data());
        if (ms != TPERM_OK) {
            std::printf("index map failed (%d) at iteration %d\n", (int)ms, it);
            return 1;
        }
        std::vector<char> seen((size_t)vol, 0);
        for (int64_t i = 0; i < vol; ++i) {
            if (map[(size_t)i] < 0 || map[(size_t)i] >= vol || seen[(size_t)map[(size_t)i]]) {
                std::printf("not a bijection at iteration %d\n", it);
                return 1;
            }
            seen[(size_t)map[(size_t)i]] = 1;
        }
        // accumulation: nontemporal loads and stores or cached, the latter from odd base pointers and
        // with line-aligned windows
        for (int pol = 1; pol <= 4; ++pol) {
            tperm::Plan q = *p;
            q.cache_policy = pol;
            if (tperm::tile_launch_policy(q, true, true) != (pol == 2 && !q.align_out ? 2 : 1) ||
                tperm::tile_launch_policy(q, true, false) != 1) {
                std::printf("an accumulating run takes the wrong cache policy, iteration %d\n", it);
                return 1;
            }
        }
        // what is read again stays in the caches, unless the caller chose the policy (these tensors are small)
        for (int pol = 0; pol <= 4; ++pol) {
            tperm_plan_opts_t with = o;
            with.cache_policy = pol;
            tperm::Plan* q = nullptr;
            if (it % 8 != 0 || tperm::create_plan(&q, rank, dims, perm, elem, &with) != TPERM_OK) break;
            const int as_planned = tperm::tile_launch_policy(*q, false, true), again = tperm::tile_launch_policy(*q, false, true, true);
            const bool cached = pol == 0 && q->cache_policy != 3;
            delete q;
            if (again != (cached ? 1 : as_planned)) {
                std::printf("the self-checking execute takes the wrong cache policy, iteration %d\n", it);
                return 1;
            }
        }
        if (p->use_lds && !p->align_out && p->tile.n_tile_dims > 0) {
            // The index map must refuse an image that ends one element too early: shrink it to what
            // the tile's first (full) instance needs and by one more.
            const tperm::TileDesc& d = p->tile;
            uint32_t last = 0;
            for (uint32_t k = 0; k < d.tile_vol; ++k)
                last = std::max(last, tperm::tile_slot(d.in_order, d.n_tile_dims, k).loff + (d.vec2 ? 1u : 0u));
            const uint32_t behind = p->spare ? 1u : 0u;
            tperm::Plan cut = *p;
            cut.tile.lds_elems = last + 1u + behind;
            const tperm_status_t fits = tperm::index_map(cut, map.data());
            cut.tile.lds_elems = last + behind;
            const bool unpadded = last + 1u == d.tile_vol * (d.vec2 ? 2u : 1u);
            if (fits != TPERM_OK || tperm::index_map(cut, map.data()) != TPERM_ERR_INTERNAL ||
                (unpadded && d.lds_elems != last + 1u + behind)) {
                std::printf("an image that is too small passes, or one is too large, iteration %d\n", it);
                return 1;
            }
            ++images;
        }
        if (p->kclass == TPERM_KERNEL_ROWCOPY || p->kclass == TPERM_KERNEL_TILED || p->kclass == TPERM_KERNEL_PACKED) {
            // the analytical model walks sampled tiles with the kernel's arithmetic: its byte
            // count per tile can never exceed the tile, and the estimate must be finite
            tperm_model_t m;
            if (tperm::model_plan(*p, &m) != TPERM_OK || !(m.microseconds > 0.0) || !(m.microseconds < 1e12) ||
                m.useful_bytes_per_tile > (double)p->cand.tile_vol * (double)elem + 0.5) {
                std::printf("model failed at iteration %d\n", it);
                return 1;
            }
        }
        if (p->align_out) ++windows;
        if (p->align_out && p->vec2) ++pair_windows;
        delete p;
        ++made;
    }
    // 253 and 262 MB in runs of 12 and 16 bytes, 144 MB in runs of two lines and in runs a little longer
    {
        struct { int64_t dims[3]; size_t elem; bool lines; } const large[] = {
            {{3, 6117, 3450}, 4, false}, {{2, 4372, 3744}, 8, false}, {{64, 640, 880}, 4, true}, {{66, 640, 880}, 4, false}, {{32, 640, 880}, 8, true}};
        const int perm[3] = {0, 2, 1};
        for (const auto& c : large) {
            tperm::Product p;
            if (tperm::build_product(&p, 3, c.dims, perm, 2, 9, c.elem, 0, 0) != TPERM_OK || p.d.out_bytes <= tperm::kCachedOutBytes ||
                tperm::nontemporal_out(p, 1 << 20) != c.lines || tperm::nontemporal_out(p, (1 << 20) + 64)) {
                std::printf("nontemporal accesses to a destination in runs of %d elements\n", (int)c.dims[0]);
                return 1;
            }
        }
    }
    int products = 0, too_large = 0;
    const int wrong = fuzz_products(2 * iters, &products, &too_large);
    if (wrong != 0) {
        std::printf("a product's plan is wrong, iteration %d\n", wrong);
        return 1;
    }
    std::printf("ok: %d plans checked (%d with line-aligned windows, %d of them in pairs, %d LDS images cut), %d option sets rejected; %d products, %d too large\n", made,
                windows, pair_windows, images, rejected, products, too_large);
    return 0;
}
