// Matrix product added straight into a permuted tensor: out[pos(i, j)] += sum_k L(i, k) R(k, j), the
// last two steps of a contraction (product, accumulating transpose) in one kernel.  pos(i, j) splits
// into a part of i and a part of j, each a sum of digits times strides of the destination.
//
// What it saves: the product is neither written nor read again (two of the four passes over a tensor
// of the destination's size), and one library call.  What bounds it: with few summed indices the
// read-modify-write of the destination (156 MB of fp64 by itself: 68 us, 4.6 TB/s), with many the matrix
// cores (4096^3: 57 TFLOP/s fp64, 129 fp32).  Measured on MI355X against the library product and the
// accumulating transpose: fp64, 11264 x 1728, K = 70 into a rank-7 tensor 155 -> 84 us; fp32 105 -> 37.
//
// Layout: workgroups of four wavefronts stay resident (three to a compute unit) and take tile after
// tile of their XCD's share.  The panels of both operands go through registers into one of two LDS
// images, kDepth summed indices at a time, and the next stage's loads travel while the matrix cores
// work on this one; the old values of the destination are requested behind the last stage's panels
// (requested earlier, the in-order memory counter makes the panels wait for them: 96 -> 86 us on the
// fp64 case above), and the next tile's first panels during the last stage.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace tperm {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
// Lane offset beyond every tensor that is accepted: the buffer range check drops the access.
constexpr uint32_t kDropped = 0xFFFFFF00u;

template <typename T> struct Mfma;
template <> struct Mfma<double> {
    typedef double acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mul(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    // row of the 16 x 16 result that element v of a lane in quarter q holds
    static __device__ __forceinline__ uint32_t row(uint32_t q, uint32_t v) { return 4u * v + q; }
};
template <> struct Mfma<float> {
    typedef float acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mul(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ uint32_t row(uint32_t q, uint32_t v) { return 4u * q + v; }
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t whole(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// N elements at a byte offset, moved with accesses of up to 16 bytes.
template <typename T, int N, int NT = 0> struct Run {
    static constexpr int kWords = N * (int)sizeof(T) / 4;
    T e[N];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
        uint32_t w[kWords];
        if constexpr (kWords >= 4) {
#pragma unroll
            for (int i = 0; i < kWords; i += 4) {
                const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff + 4 * i, (int)soff, NT);
                w[i] = x.x, w[i + 1] = x.y, w[i + 2] = x.z, w[i + 3] = x.w;
            }
        } else if constexpr (kWords == 2) {
            const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, NT);
            w[0] = x.x, w[1] = x.y;
        } else {
            w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, NT);
        }
        __builtin_memcpy(e, w, sizeof(e));
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t voff) const {
        uint32_t w[kWords];
        __builtin_memcpy(w, e, sizeof(e));
        if constexpr (kWords >= 4) {
#pragma unroll
            for (int i = 0; i < kWords; i += 4) __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[i], w[i + 1], w[i + 2], w[i + 3]}, r, (int)voff + 4 * i, 0, NT);
        } else if constexpr (kWords == 2) {
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, r, (int)voff, 0, NT);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(w[0], r, (int)voff, 0, NT);
        }
    }
};

// One operand's panel of FREE x kDepth elements, from global memory through registers to LDS, where
// it lies with the free index running fastest (pitch kPitch).  K_FIRST: the summed index is the
// stride-1 one in memory.
template <typename T, int FREE, bool K_FIRST> struct Panel {
    // elements per load: 16 bytes, less where the panel has too few for all threads
    static constexpr int V = FREE * kDepth / kThreads < 16 / (int)sizeof(T) ? FREE * kDepth / kThreads : 16 / (int)sizeof(T);
    static constexpr int kPasses = FREE * kDepth / (kThreads * V);
    static_assert(kPasses * kThreads * V == FREE * kDepth, "whole passes");
    static constexpr int kAcross = (K_FIRST ? kDepth : FREE) / V;   // vectors along the stride-1 index
    static constexpr int kPitch = FREE + 16 / (int)sizeof(T);
    Run<T, V> reg[kPasses];

    static __device__ __forceinline__ void place(int p, uint32_t* free, uint32_t* k) {
        const uint32_t idx = threadIdx.x + (uint32_t)p * kThreads;
        const uint32_t along = idx % (uint32_t)kAcross * V, other = idx / (uint32_t)kAcross;
        *free = K_FIRST ? other : along;
        *k = K_FIRST ? along : other;
    }
    // the panel at (f0, k0) of a tensor of n x depth elements
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t n, uint32_t depth, uint32_t f0, uint32_t k0) {
        const uint32_t soff = (K_FIRST ? k0 + depth * f0 : f0 + n * k0) * (uint32_t)sizeof(T);
        // Vectors along the free index may run past its end wherever another row follows: what they
        // fetch there reaches rows and columns of the result that do not exist.  The summed index has to
        // end exactly.
        if (K_FIRST ? k0 + kDepth <= depth : f0 + FREE <= n || (k0 + kDepth < depth && n >= (uint32_t)V)) {
#pragma unroll
            for (int p = 0; p < kPasses; ++p) {
                uint32_t f, k;
                place(p, &f, &k);
                const bool there = f0 + f < n && (K_FIRST || k0 + k < depth);
                reg[p].load(r, there ? (K_FIRST ? k + depth * f : f + n * k) * (uint32_t)sizeof(T) : kDropped, soff);
            }
        } else {
            // the end of the stride-1 index: element by element, zero beyond it
#pragma unroll
            for (int p = 0; p < kPasses; ++p) {
                uint32_t f, k;
                place(p, &f, &k);
                const uint32_t at = (K_FIRST ? k + depth * f : f + n * k) * (uint32_t)sizeof(T);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const bool there = f0 + f + (K_FIRST ? 0u : (uint32_t)i) < n && k0 + k + (K_FIRST ? (uint32_t)i : 0u) < depth;
                    Run<T, 1> one;
                    one.load(r, there ? at + (uint32_t)i * (uint32_t)sizeof(T) : kDropped, soff);
                    reg[p].e[i] = one.e[0];
                }
            }
        }
    }
    __device__ __forceinline__ void put(T* lds) const {
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            uint32_t f, k;
            place(p, &f, &k);
            if constexpr (K_FIRST) {
#pragma unroll
                for (int i = 0; i < V; ++i) lds[(k + i) * kPitch + f] = reg[p].e[i];
            } else {
                __builtin_memcpy(__builtin_assume_aligned(lds + k * kPitch + f, V * sizeof(T)), reg[p].e, V * sizeof(T));
            }
        }
    }
};

// Tile shapes: CB x RB blocks of 16 x 16 to a wavefront, four wavefronts, WAVES_FAST of them side by
// side along the fast index.
template <int CB_, int RB_, int WAVES_FAST> struct Shape {
    static constexpr int CB = CB_, RB = RB_, kWavesFast = WAVES_FAST;
    static constexpr int TF = WAVES_FAST * 16 * CB, TS = kThreads / 64 / WAVES_FAST * 16 * RB;
};
template <typename T> struct Shapes;
template <> struct Shapes<double> {
    typedef Shape<4, 1, 2> wide;       // 128 x 32
    typedef Shape<1, 2, 1> thin_fast;  // 16 x 128
    typedef wide thin_slow;
};
template <> struct Shapes<float> {
    typedef Shape<4, 2, 2> wide;       // 128 x 64
    typedef Shape<1, 4, 1> thin_fast;  // 16 x 256
    typedef Shape<4, 1, 4> thin_slow;  // 256 x 16
};

template <typename T, typename S, bool FAST_K, bool SLOW_K, int VEC, int NT, bool SPLIT>
__global__ void __launch_bounds__(kThreads, kResident)
product_kernel(const ProductDesc d, const T* __restrict__ fast, const T* __restrict__ slow, T* __restrict__ out) {
    static_assert(!SPLIT || (VEC == 1 && NT == 0), "one form writes partial products");
    constexpr int CB = S::CB, RB = S::RB, TF = S::TF, TS = S::TS;
    typedef Panel<T, TF, FAST_K> FastPanel;
    typedef Panel<T, TS, SLOW_K> SlowPanel;
    typedef Mfma<T> mfma;
    __shared__ __align__(16) T lds_f[2][kDepth * FastPanel::kPitch];
    __shared__ __align__(16) T lds_s[2][kDepth * SlowPanel::kPitch];
    __shared__ uint32_t off[2][TF + TS];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t c = lane & 15u, q = lane >> 4;
    const uint32_t wf = wave % S::kWavesFast * (16u * CB), ws = wave / S::kWavesFast * (16u * RB);
    const __amdgpu_buffer_rsrc_t rf = whole(fast, d.fast_bytes), rs = whole(slow, d.slow_bytes), ro = whole(out, d.out_bytes);
    // the tiles of this workgroup: every step-th of its XCD's share
    const uint32_t first = (blockIdx.x & 7u) * d.per_xcd, tiles = d.tiles_fast * d.tiles_slow, all = SPLIT ? tiles * d.splits : tiles;
    const uint32_t end = first + d.per_xcd < all ? first + d.per_xcd : all, hop = gridDim.x >> 3;
    uint32_t t = first + (blockIdx.x >> 3);
    if (t >= end) return;

    FastPanel pf;
    SlowPanel ps;
    uint32_t f0, s0, k_begin = 0, k_end = d.k, buf = 0, table = 0;
    auto locate = [&](uint32_t unit) {
        const uint32_t tile = SPLIT ? unit % tiles : unit;
        f0 = tile / d.tiles_slow * TF, s0 = tile % d.tiles_slow * TS;
        if (SPLIT) {
            k_begin = unit / tiles * d.k_split;
            k_end = k_begin + d.k_split < d.k ? k_begin + d.k_split : d.k;
        }
    };
    auto fetch = [&](uint32_t k0) {
        pf.load(rf, d.n_fast, d.k, f0, k0);
        ps.load(rs, d.n_slow, d.k, s0, k0);
    };
    auto put = [&]() {
        pf.put(lds_f[buf]);
        ps.put(lds_s[buf]);
    };
    // byte offsets of the tile's rows and columns in the destination
    auto tabulate = [&]() {
        if (SPLIT) return;
        for (uint32_t e = tid; e < TF + TS; e += kThreads) {
            const bool is_f = e < TF;
            const uint32_t i = is_f ? f0 + e : s0 + e - TF;
            const ProductDim* dim = is_f ? d.fast : d.slow;
            uint32_t rem = i, at = 0;
            for (uint32_t z = 0; z < (is_f ? d.fast_dims : d.slow_dims); ++z) {
                const uint32_t quot = fdiv(rem, dim[z].div);
                at += (rem - quot * dim[z].ext) * dim[z].stride;
                rem = quot;
            }
            off[table][e] = i < (is_f ? d.n_fast : d.n_slow) ? at : kDropped;
        }
    };
    locate(t);
    fetch(k_begin);
    tabulate();
    put();
    __syncthreads();

    // position of block cb's element of this lane along the fast index: VEC neighbours to a lane, so that
    // the sixteen lanes of a row reach whole stretches of the destination with one access
    auto col = [&](int cb) { return (uint32_t)(cb / VEC) * (16u * VEC) + VEC * c + (uint32_t)(cb % VEC); };
    typename mfma::acc acc[CB][RB];
    auto step = [&](uint32_t k) {
        T f[CB], s[RB];
        const uint32_t row = k + q;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) f[cb] = lds_f[buf][row * FastPanel::kPitch + wf + col(cb)];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) s[rb] = lds_s[buf][row * SlowPanel::kPitch + ws + RB * c + rb];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[cb][rb] = mfma::mul(s[rb], f[cb], acc[cb][rb]);
    };
    static_assert(CB % VEC == 0, "whole stretches");
    constexpr int G = CB / VEC;
    auto place = [&](uint32_t of, uint32_t os) { return of == kDropped || os == kDropped ? kDropped : of + os; };
    for (;;) {
        const uint32_t* off_f = off[table] + wf;
        const uint32_t* off_s = off[table] + TF + ws;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[cb][rb] = typename mfma::acc{0, 0, 0, 0};
        const uint32_t end_k = k_end, last = k_begin + (k_end - k_begin - 1u) / kDepth * kDepth;
        auto stage = [&]() {
#pragma unroll
            for (uint32_t k = 0; k < kDepth; k += 4) step(k);
            buf ^= 1u;
            put();
            __syncthreads();
        };
        const bool more = last > k_begin;
        for (uint32_t k0 = k_begin + kDepth; k0 < last; k0 += kDepth) {
            fetch(k0);
            stage();
        }
        if (more) fetch(last);
        // what the destination holds: fetched behind the last panels, needed after the last step
        Run<T, VEC, NT> old[RB][4][G];
        if constexpr (!SPLIT)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int g = 0; g < G; ++g) old[rb][v][g].load(ro, place(off_f[col(g * VEC)], off_s[mfma::row(q, v) * RB + rb]), 0);
        if (more) stage();
        // the last stage; the next tile's first panels travel meanwhile
        const uint32_t next = t + hop;
        if (next < end) {
            locate(next);
            fetch(k_begin);
        }
        for (uint32_t k = 0; last + k < end_k; k += 4) step(k);
        if constexpr (SPLIT) {
            T* part = out + (size_t)t * (TF * TS) + tid;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) part[((rb * 4 + v) * CB + cb) * kThreads] = acc[cb][rb][v];
        } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    Run<T, VEC, NT> sum;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) sum.e[e] = old[rb][v][g].e[e] + acc[g * VEC + e][rb][v];
                    sum.store(ro, place(off_f[col(g * VEC)], off_s[mfma::row(q, v) * RB + rb]));
                }
        }
        if (next >= end) break;
        t = next;
        buf ^= 1u;
        table ^= 1u;
        put();
        tabulate();
        __syncthreads();
    }
}

// Adds up the partial products of a tile, in the order of the summed index, and adds the total to the
// destination: one workgroup per tile and register of the kernel above, whose layout the partials have.
template <typename T, typename S>
__global__ void __launch_bounds__(kThreads)
product_sum_kernel(const ProductDesc d, const T* __restrict__ part, T* __restrict__ out) {
    constexpr uint32_t TF = S::TF, TS = S::TS, CB = S::CB, RB = S::RB, kRegs = 4u * CB * RB;
    const uint32_t tile = blockIdx.x / kRegs, reg = blockIdx.x % kRegs;
    const uint32_t rb = reg / (4u * CB), v = reg / CB % 4u, cb = reg % CB;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, c = lane & 15u, q = lane >> 4;
    const uint32_t f = tile / d.tiles_slow * TF + wave % S::kWavesFast * (16u * CB) + 16u * cb + c;
    const uint32_t s = tile % d.tiles_slow * TS + wave / S::kWavesFast * (16u * RB) + Mfma<T>::row(q, v) * RB + rb;
    if (f >= d.n_fast || s >= d.n_slow) return;
    uint32_t at = 0, rem = f;
    for (uint32_t z = 0; z < d.fast_dims; ++z) {
        const uint32_t quot = fdiv(rem, d.fast[z].div);
        at += (rem - quot * d.fast[z].ext) * d.fast[z].stride;
        rem = quot;
    }
    rem = s;
    for (uint32_t z = 0; z < d.slow_dims; ++z) {
        const uint32_t quot = fdiv(rem, d.slow[z].div);
        at += (rem - quot * d.slow[z].ext) * d.slow[z].stride;
        rem = quot;
    }
    T* to = reinterpret_cast<T*>(reinterpret_cast<char*>(out) + at);
    const T old = *to;
    const size_t step = (size_t)d.tiles_fast * d.tiles_slow * (TF * TS);
    const T* p = part + (size_t)tile * (TF * TS) + reg * kThreads + tid;
    T sum = 0;
#pragma unroll 8
    for (uint32_t i = 0; i < d.splits; ++i) sum += p[i * step];
    *to = old + sum;
}

template <typename T, typename S, bool FAST_K, bool SLOW_K>
static const void* product_ptr(const Product& p, const void* out) {
#define TPERM_PRODUCT(VEC, NT, SPLIT) reinterpret_cast<const void*>(&product_kernel<T, S, FAST_K, SLOW_K, VEC, NT, SPLIT>)
    if (p.d.splits > 1u) return TPERM_PRODUCT(1, 0, true);
    if constexpr (S::CB == 1) {
        return TPERM_PRODUCT(1, 0, false);
    } else {
        // runs of whole lines hold whole 16-byte accesses
        if (nontemporal_out(p, reinterpret_cast<uintptr_t>(out))) return TPERM_PRODUCT(16 / (int)sizeof(T), 2, false);
        if constexpr (sizeof(T) == 4)
            if (p.vec == 4) return TPERM_PRODUCT(4, 0, false);
        return p.vec >= 2 ? TPERM_PRODUCT(2, 0, false) : TPERM_PRODUCT(1, 0, false);
    }
#undef TPERM_PRODUCT
}

template <typename T, typename S>
static hipError_t launch_shape(const Product& p, const void* left, const void* right, void* out, void* workspace, int num_cu, hipStream_t stream) {
    const void* f = p.fast_k_first ? (p.slow_k_first ? product_ptr<T, S, true, true>(p, out) : product_ptr<T, S, true, false>(p, out))
                                   : (p.slow_k_first ? product_ptr<T, S, false, true>(p, out) : product_ptr<T, S, false, false>(p, out));
    ProductDesc d = p.d;
    const void* fast = p.left_fast ? left : right;
    const void* slow = p.left_fast ? right : left;
    void* to = d.splits > 1u ? workspace : out;
    void* args[] = {(void*)&d, (void*)&fast, (void*)&slow, (void*)&to};
    const uint32_t per = ((uint32_t)num_cu * kResident + 7u) / 8u;  // resident workgroups of one XCD
    hipError_t err = hipLaunchKernel(f, dim3(8u * (d.per_xcd < per ? d.per_xcd : per)), dim3(kThreads), args, 0, stream);
    if (err != hipSuccess || d.splits == 1u) return err;
    hipLaunchKernelGGL((product_sum_kernel<T, S>), dim3(d.tiles_fast * d.tiles_slow * 4u * S::CB * S::RB), dim3(kThreads), 0, stream, d, (const T*)workspace, (T*)out);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_type(const Product& p, const void* left, const void* right, void* out, void* workspace, int num_cu, hipStream_t stream) {
    switch (p.shape) {
        case 1: return launch_shape<T, typename Shapes<T>::thin_fast>(p, left, right, out, workspace, num_cu, stream);
        case 2: return launch_shape<T, typename Shapes<T>::thin_slow>(p, left, right, out, workspace, num_cu, stream);
        default: return launch_shape<T, typename Shapes<T>::wide>(p, left, right, out, workspace, num_cu, stream);
    }
}

hipError_t launch_product(const Product& p, const void* left, const void* right, void* out, void* workspace, int num_cu, hipStream_t stream) {
    return p.elem == 8 ? launch_type<double>(p, left, right, out, workspace, num_cu, stream)
                       : launch_type<float>(p, left, right, out, workspace, num_cu, stream);
}

}  // namespace tperm
