// On-device multiset check behind tperm_execute_verified: after a transpose, the output must
// hold exactly the elements of the input, each as often (a transpose moves bits and creates or
// destroys none of them).  Three order-independent digests of the element words -- their sum
// and their exclusive-or, and the sum of a scrambled image of every word, all modulo 2^64 --
// are computed for both tensors and compared on the device.
//
// Work layout: both tensors are cut into chunks of kVerifyChunk elements; one workgroup digests one
// chunk and writes one partial result (32 bytes) into a scratch buffer, the first tensor's chunks in
// the slots 0 to chunks - 1 and the second's behind them; a last, single workgroup adds up the
// differences of the two tensors' partials and writes the verdict.  Every slot that is read has been
// written by the same call, so the scratch needs no clearing.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "verify.hpp"

// Scratch of the entry point that allocates nothing: one copy of this array lives on every GPU
// the library runs on, from the moment its code is loaded there until the process ends.  Host
// code never passes the array's name to a kernel (on the host that name is only a handle for
// the symbol): verify_static_scratch() asks the runtime for the array's device address, once per
// device, and every kernel argument is built from that address.
static __device__ __align__(256) unsigned char scratch[tperm::kVerifyStaticBytes];

namespace tperm {

struct MultisetPartial {
    uint64_t sum, exor, mix, unused;
};
static_assert(sizeof(MultisetPartial) == kVerifyPartialBytes, "partial result size");

// A chunk is digested by 1024 threads with all their 16-byte loads (four or eight each) in flight
// at once.  What bounds it: memory for large tensors; one round trip to memory plus the reductions
// for small ones.  Measured on MI355X (sums across lanes by shuffles, see Triple), both tensors of a transpose just made (by tperm_execute; behind the
// cached step of tperm_execute_verified 44 instead of 49), with the verdict, in microseconds (with one word per load, a workgroup of 256 threads and a launch per tensor before):
// 2 x 134 MB of 4-byte words 49 (96), 2 x 500 MB 171 (343), 2 x 0.26 MB 7.5 (41); 8-byte words 49 (91),
// 169 (215), 8.5 (43).  512 threads are level on large tensors, 256 are up to 10 % behind.
constexpr int kPartialThreads = 1024;
constexpr int kVerdictThreads = 1024;

// What is summed of every word: the word times an odd constant, its high half folded into its low
// half.  A word and its image share no linear relation, so two corrupted elements whose plain sums
// and exclusive-ors happen to cancel still show.  (The scrambled sum is the sum of these images
// times a second odd constant; a factor common to all terms needs to be multiplied once, not once
// per element.)
__device__ __forceinline__ uint64_t image(uint64_t e) {
    const uint64_t h = e * 0x9E3779B97F4A7C15ull;
    return h ^ (h >> 29);
}
constexpr uint64_t kScrambleFactor = 0xBF58476D1CE4E5B9ull;

// One step of a sum across lanes: x of the lane that the DPP control names, 0 where there is none.
template <int CTRL>
__device__ __forceinline__ uint64_t from_lane(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, 0xF, 0xF, true);
    return ((uint64_t)hi << 32) | lo;
}

// Totals of three values over 16 lanes, in the last lane of each row, and over the wavefront, in lane 63.  In registers
// (DPP row shifts and broadcasts): through the LDS (shuffles), the sixteen wavefronts of a workgroup queue for
// 36 passes each: 2 x 0.2 to 2.1 MB 4.5 to 5.0 us against 3.6 to 4.1 for the digests, 3.0 against 1.7 for the verdict; on
// tensors of 134 MB the kernels by themselves take the same.  Self-checking execute with shuffles / with these, in
// microseconds: 2 x 0.23 MB 11.7 / 9.6, 2 x 2.1 MB 10.8 / 8.8, 2 x 24 MB 26.4 / 24.4, 2 x 64 MB 51.2 / 49.3, 2 x 159 MB 129.9 / 127.1.
struct Triple {
    uint64_t s, x, m;
    template <int CTRL> __device__ __forceinline__ void step() {
        s += from_lane<CTRL>(s);
        x ^= from_lane<CTRL>(x);
        m += from_lane<CTRL>(m);
    }
    __device__ __forceinline__ void row_total() {
        step<0x111>();  // row_shr:1, 2, 4, 8
        step<0x112>();
        step<0x114>();
        step<0x118>();
    }
    __device__ __forceinline__ void wave_total() {
        row_total();
        // lane 15 of a row into the row after it, then lane 31 into the upper half (other rows get values of no use)
        step<0x142>();
        step<0x143>();
    }
};

// Adds up three 64-bit values over the threads of a workgroup of at most 16 wavefronts; the totals end up in
// every thread of its first wavefront.
template <int THREADS>
__device__ __forceinline__ void block_reduce3(uint64_t* s, uint64_t* x, uint64_t* m) {
    constexpr uint32_t kWaves = THREADS / 64;
    static_assert(kWaves >= 1 && kWaves <= 16, "one row of lanes adds up the wavefronts");
    __shared__ uint64_t red[3][kWaves];
    Triple t = {*s, *x, *m};
    t.wave_total();
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    if (lane == 63u) {
        red[0][wave] = t.s;
        red[1][wave] = t.x;
        red[2][wave] = t.m;
    }
    __syncthreads();
    if (wave == 0) {
        t = {lane < kWaves ? red[0][lane] : 0, lane < kWaves ? red[1][lane] : 0, lane < kWaves ? red[2][lane] : 0};
        t.row_total();
        auto total = [](uint64_t v) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 15), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 15);
            return ((uint64_t)hi << 32) | lo;
        };
        *s = total(t.s);
        *x = total(t.x);
        *m = total(t.m);
    }
}

// Sixteen bytes of words, loaded at once from an address aligned to one word.
template <typename T> struct WordVec {
    static constexpr uint32_t kWords = 16 / sizeof(T);
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4)));
    static __device__ __forceinline__ uint64_t word(const type& v, uint32_t i) {
        return sizeof(T) == 4 ? (uint64_t)v[i] : ((uint64_t)v[2 * i + 1] << 32) | v[2 * i];
    }
};

// One workgroup per chunk of kVerifyChunk elements, both tensors in one launch; T is the element word.
template <typename T>
__global__ void __launch_bounds__(kPartialThreads)
multiset_partial_kernel(const T* __restrict__ a, const T* __restrict__ b, uint64_t n, uint32_t chunks,
                        MultisetPartial* __restrict__ partial) {
    constexpr uint32_t V = WordVec<T>::kWords, kStep = kPartialThreads * V;
    constexpr uint32_t kLoads = (uint32_t)kVerifyChunk / kStep;
    static_assert(kVerifyChunk % kStep == 0, "whole rounds of vector loads per chunk");
    // last chunks first: the end of the tensor that was written last is what the last-level cache holds
    const uint32_t slot = 2u * chunks - 1u - blockIdx.x;
    const bool second = slot >= chunks;
    const uint64_t begin = (uint64_t)(second ? slot - chunks : slot) * kVerifyChunk;
    const T* p = (second ? b : a) + begin;
    uint64_t s = 0, x = 0, m = 0;
    auto take = [&](uint64_t e) {
        s += e;
        x ^= e;
        m += image(e);
    };
    typedef WordVec<T> vec;
    auto load = [&](uint32_t i) { return *reinterpret_cast<const typename vec::type*>(p + i); };
    auto take_vec = [&](const typename vec::type& v) {
#pragma unroll
        for (uint32_t i = 0; i < V; ++i) take(vec::word(v, i));
    };
    if (begin + kVerifyChunk <= n) {
        typename vec::type v[kLoads];
#pragma unroll
        for (uint32_t j = 0; j < kLoads; ++j) v[j] = load(j * kStep + threadIdx.x * V);
#pragma unroll
        for (uint32_t j = 0; j < kLoads; ++j) take_vec(v[j]);
    } else {
        // the short last chunk: the vectors it lacks read its start instead and count as zero,
        // which is neutral to all three digests
        const uint32_t left = (uint32_t)(n - begin), odd = left % V;
        if (left >= V) {
#pragma unroll 4
            for (uint32_t j = 0; j < kLoads; ++j) {
                const uint32_t i = j * kStep + threadIdx.x * V;
                const bool there = i + V <= left;
                typename vec::type v = load(there ? i : 0u);
                if (!there) v = 0u;
                take_vec(v);
            }
        }
        if (threadIdx.x < odd) take((uint64_t)p[left - odd + threadIdx.x]);
    }
    block_reduce3<kPartialThreads>(&s, &x, &m);
    if (threadIdx.x == 0) {
        MultisetPartial r;
        r.sum = s;
        r.exor = x;
        r.mix = m * kScrambleFactor;
        r.unused = 0;
        partial[slot] = r;
    }
}

// Single workgroup: the partials of the two tensors, subtracted and added up.  *verdict = 0 when all
// three digests agree, else a bit mask of the ones that differ (1 sum, 2 exclusive-or, 4 scrambled sum).
__global__ void __launch_bounds__(kVerdictThreads)
multiset_verdict_kernel(const MultisetPartial* __restrict__ pa, const MultisetPartial* __restrict__ pb,
                        uint32_t chunks, uint64_t* __restrict__ verdict) {
    uint64_t s = 0, x = 0, m = 0;
#pragma unroll 4
    for (uint32_t c = threadIdx.x; c < chunks; c += kVerdictThreads) {
        s += pa[c].sum - pb[c].sum;
        x ^= pa[c].exor ^ pb[c].exor;
        m += pa[c].mix - pb[c].mix;
    }
    block_reduce3<kVerdictThreads>(&s, &x, &m);
    if (threadIdx.x == 0) *verdict = (s != 0 ? 1u : 0u) | (x != 0 ? 2u : 0u) | (m != 0 ? 4u : 0u);
}

hipError_t verify_static_scratch(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mutex;
    static void* address[kMaxDevices] = {};  // per device ordinal; nullptr = not asked yet
    *ptr = nullptr;
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mutex);
    if (address[dev] == nullptr) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // the current device's copy
        if (err != hipSuccess) return err;
        if (p == nullptr) return hipErrorInvalidSymbol;
        address[dev] = p;
    }
    *ptr = address[dev];
    return hipSuccess;
}

size_t verify_scratch_bytes(uint64_t n_elems) {
    const uint64_t chunks = (n_elems + kVerifyChunk - 1) / kVerifyChunk;
    return (size_t)(2 * chunks * kVerifyPartialBytes);
}

hipError_t launch_multiset_compare(const void* a, const void* b, uint64_t n_elems, int elem,
                                   void* scratch_dev, uint64_t* verdict_dev, hipStream_t stream) {
    const uint64_t chunks64 = (n_elems + kVerifyChunk - 1) / kVerifyChunk;
    if (chunks64 == 0 || chunks64 > 0x3FFFFFFFull) return hipErrorInvalidValue;
    const uint32_t chunks = (uint32_t)chunks64;
    MultisetPartial* pa = static_cast<MultisetPartial*>(scratch_dev);
    MultisetPartial* pb = pa + chunks;
    const dim3 grid(2u * chunks);
    if (elem == 8)
        hipLaunchKernelGGL(multiset_partial_kernel<uint64_t>, grid, dim3(kPartialThreads), 0, stream,
                           static_cast<const uint64_t*>(a), static_cast<const uint64_t*>(b), n_elems, chunks, pa);
    else
        hipLaunchKernelGGL(multiset_partial_kernel<uint32_t>, grid, dim3(kPartialThreads), 0, stream,
                           static_cast<const uint32_t*>(a), static_cast<const uint32_t*>(b), n_elems, chunks, pa);
    hipLaunchKernelGGL(multiset_verdict_kernel, dim3(1), dim3(kVerdictThreads), 0, stream, pa, pb, chunks, verdict_dev);
    return hipGetLastError();
}

}  // namespace tperm
