// Canonical order of a candidate list: ascending CL1 word (row, then plane,
// then bin), i.e. a stable sort of the 8-byte entries on their low 32 bits
// (the power in the high half travels with its word).
//
// Up to kSortMax entries: the list is parted into up to 8192 buckets of equal
// width (a power of two) between its smallest and largest word, each entry
// with its place in the input, and every bucket is ordered on its own by
// counting, for each entry, the entries before it.  Words are unique and
// spread over rows, planes and bins, so buckets hold tens to a few hundred
// entries (plane 1 has the most); (word, place) is unique, so the order
// inside a bucket does not matter and equal words keep their order.
//   1. k_sort_range    smallest and largest word per block;
//   2. k_sort_hist     bucket counts per block;
//   3. k_sort_scan     per bucket, the counts of the blocks before each;
//   4. k_sort_scatter  entries to their buckets (blocks in order);
//   5. k_sort_buckets  one wave per bucket.
// A list of at most kSortOne entries takes one block for 1-4.  All are bound
// by latency and scattered stores (a few MB in the L2), so few passes win:
// 305 K entries 112 us as nine rocPRIM launches, 58 us so (4 + 5 + 6 + 17 +
// 26); 7 K entries 18 us as three, 15 us as two.  Longer lists go to
// rocPRIM, which large passes suit.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>

#include <type_traits>

#include "hs_internal.h"

namespace hsk {

namespace {

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int64_t kSortMax = (int64_t)1 << 20;
constexpr int64_t kSortOne = 16384;
constexpr int kSTh = 1024;              // threads of the passes over the list
constexpr int kSortBlocks = 128;
constexpr int kSU = 4;                  // loads in flight per thread
constexpr int kBinsMax = 8192;
constexpr int kBucket = 1024;           // entries of a bucket ordered in LDS

int sort_blocks(int64_t n)
{
    const int64_t b = (n + (int64_t)kSTh * kSU - 1) / ((int64_t)kSTh * kSU);
    return (int)(b < 1 ? 1 : (b > kSortBlocks ? kSortBlocks : b));
}

// Buckets of a list: about 32 entries in the mean (plane 1 of the survey's
// thresholds holds half of all candidates in an eighth of the words).
int sort_bins(int64_t n)
{
    int b = 64;
    while (b < kBinsMax && (int64_t)b * 32 < n) b *= 2;
    return b;
}

struct Range {
    uint32_t lo, hi;
};

__device__ __forceinline__ int bin_shift(const Range& r, int bins)
{
    const uint32_t span = r.hi - r.lo;
    const int need = span == 0 ? 0 : 32 - __builtin_clz(span);      // bits of span
    const int have = 31 - __builtin_clz((uint32_t)bins);
    return need > have ? need - have : 0;
}

__device__ __forceinline__ void chunk(int64_t n, int64_t& e0, int64_t& e1)
{
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    e0 = (int64_t)blockIdx.x * per;
    e1 = e0 + per < n ? e0 + per : n;
    if (e0 > n) e0 = n;
}

// f(entry, place) for the entries of [e0, e1), kSU loads in flight per thread.
template <typename F>
__device__ __forceinline__ void each(const uint64_t* __restrict__ a, int64_t e0, int64_t e1, F f)
{
    for (int64_t b = e0 + threadIdx.x; b < e1; b += (int64_t)kSU * kSTh) {
        uint64_t x[kSU];
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
            const int64_t e = b + (int64_t)u * kSTh;
            x[u] = a[e < e1 ? e : e1 - 1];
        }
#pragma unroll
        for (int u = 0; u < kSU; ++u)
            if (b + (int64_t)u * kSTh < e1) f(x[u], (uint32_t)(b + (int64_t)u * kSTh));
    }
}

// Smallest and largest of the block's (lo, hi); every thread gets it.
__device__ __forceinline__ Range block_range(uint32_t lo, uint32_t hi)
{
    __shared__ Range part[kSTh / 64];
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t l = (uint32_t)__shfl_xor((int)lo, d, 64), h = (uint32_t)__shfl_xor((int)hi, d, 64);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = Range{lo, hi};
    __syncthreads();
    Range r = part[0];
    for (int w = 1; w < kSTh / 64; ++w) {
        r.lo = part[w].lo < r.lo ? part[w].lo : r.lo;
        r.hi = part[w].hi > r.hi ? part[w].hi : r.hi;
    }
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kSTh) void k_sort_range(const uint64_t* __restrict__ cand, int64_t n,
                                                     Range* __restrict__ parts)
{
    int64_t e0, e1;
    chunk(n, e0, e1);
    uint32_t lo = ~0u, hi = 0;
    each(cand, e0, e1, [&](uint64_t x, uint32_t) {
        const uint32_t w = (uint32_t)x;
        lo = w < lo ? w : lo;
        hi = w > hi ? w : hi;
    });
    const Range r = block_range(lo, hi);
    if (threadIdx.x == 0) parts[blockIdx.x] = r;
}

__device__ __forceinline__ Range whole_range(const Range* __restrict__ parts, int G)
{
    const int l = threadIdx.x & 63;                    // two blocks' ranges per lane
    Range r = parts[l < G ? l : 0];
    const Range r2 = parts[l + 64 < G ? l + 64 : 0];
    r.lo = r2.lo < r.lo ? r2.lo : r.lo;
    r.hi = r2.hi > r.hi ? r2.hi : r.hi;
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t l = (uint32_t)__shfl_xor((int)r.lo, d, 64), h = (uint32_t)__shfl_xor((int)r.hi, d, 64);
        r.lo = l < r.lo ? l : r.lo;
        r.hi = h > r.hi ? h : r.hi;
    }
    return r;
}
static_assert(kSortBlocks <= 128, "two blocks per lane");

__global__ __launch_bounds__(kSTh) void k_sort_hist(const uint64_t* __restrict__ cand, int64_t n, int bins,
                                                    const Range* __restrict__ parts, uint32_t* __restrict__ ph)
{
    __shared__ uint32_t hist[kBinsMax];
    for (int i = threadIdx.x; i < bins; i += kSTh) hist[i] = 0;
    const Range r = whole_range(parts, gridDim.x);
    const int s = bin_shift(r, bins);
    __syncthreads();
    int64_t e0, e1;
    chunk(n, e0, e1);
    each(cand, e0, e1, [&](uint64_t x, uint32_t) { atomicAdd(&hist[((uint32_t)x - r.lo) >> s], 1u); });
    __syncthreads();
    for (int i = threadIdx.x; i < bins; i += kSTh) ph[(int64_t)blockIdx.x * bins + i] = hist[i];
}

// Exclusive sum over the block's threads.
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v)
{
    __shared__ uint32_t wsum[kSTh / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    __syncthreads();
    return before + inc - v;
}

// An entry with its place in the input.
struct alignas(16) Placed {
    uint64_t e;
    uint32_t i, pad;
};

// Counts of block g and bin b to the entries of bin b in blocks before g;
// total[b]: all of them.
constexpr int kScanTh = 256;
__global__ __launch_bounds__(kScanTh) void k_sort_scan(uint32_t* __restrict__ ph, int G, int bins,
                                                       uint32_t* __restrict__ total)
{
    const int b = blockIdx.x * kScanTh + threadIdx.x;
    if (b >= bins) return;
    uint32_t at = 0;
    for (int g0 = 0; g0 < G; g0 += 16) {
        uint32_t v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = ph[(int64_t)(g0 + q < G ? g0 + q : G - 1) * bins + b];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            if (g0 + q < G) {
                ph[(int64_t)(g0 + q) * bins + b] = at;
                at += v[q];
            }
        }
    }
    total[b] = at;
}

__global__ __launch_bounds__(kSTh) void k_sort_scatter(const uint64_t* __restrict__ cand, int64_t n, int bins,
                                                       const Range* __restrict__ parts,
                                                       const uint32_t* __restrict__ ph,
                                                       const uint32_t* __restrict__ total,
                                                       uint32_t* __restrict__ start, Placed* __restrict__ out)
{
    __shared__ uint32_t cur[kBinsMax];
    const Range r = whole_range(parts, gridDim.x);
    const int s = bin_shift(r, bins);
    // each thread's run of bins: where the bin starts, plus the part of the
    // blocks before this one
    constexpr int kPer = kBinsMax / kSTh;
    const int per = bins >= kSTh ? bins / kSTh : 1;
    const int b0 = threadIdx.x * per;
    uint32_t tot[kPer], mine[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const bool in = q < per && b0 + q < bins;
        tot[q] = in ? total[b0 + q] : 0u;
        mine[q] = in ? ph[(int64_t)blockIdx.x * bins + b0 + q] : 0u;
        sum += tot[q];
    }
    uint32_t at = block_exclusive(sum);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        if (q < per && b0 + q < bins) {
            cur[b0 + q] = at + mine[q];
            if (blockIdx.x == 0) start[b0 + q] = at;
            at += tot[q];
        }
    }
    if (blockIdx.x == 0 && b0 < bins && b0 + per == bins) start[bins] = at;
    __syncthreads();
    int64_t e0, e1;
    chunk(n, e0, e1);
    each(cand, e0, e1, [&](uint64_t x, uint32_t i) {
        out[atomicAdd(&cur[((uint32_t)x - r.lo) >> s], 1u)] = Placed{x, i, 0};
    });
}

// The passes before the buckets for a short list, in one block.
__global__ __launch_bounds__(kSTh) void k_sort_one(const uint64_t* __restrict__ cand, int n, int bins,
                                                   uint32_t* __restrict__ start, Placed* __restrict__ out)
{
    __shared__ uint32_t cur[kSTh];
    constexpr int U = (int)(kSortOne / kSTh);
    uint64_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = (int)threadIdx.x + u * kSTh;
        x[u] = e < n ? cand[e] : 0;
    }
    if ((int)threadIdx.x < bins) cur[threadIdx.x] = 0;
    uint32_t lo = ~0u, hi = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t w = (uint32_t)x[u];
        if ((int)threadIdx.x + u * kSTh < n) {
            lo = w < lo ? w : lo;
            hi = w > hi ? w : hi;
        }
    }
    const Range r = block_range(lo, hi);
    const int s = bin_shift(r, bins);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if ((int)threadIdx.x + u * kSTh < n) atomicAdd(&cur[((uint32_t)x[u] - r.lo) >> s], 1u);
    __syncthreads();
    const uint32_t mine = (int)threadIdx.x < bins ? cur[threadIdx.x] : 0u;
    const uint32_t at = block_exclusive(mine);
    if ((int)threadIdx.x < bins) {
        cur[threadIdx.x] = at;
        start[threadIdx.x] = at;
        if ((int)threadIdx.x == bins - 1) start[bins] = at + mine;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = (int)threadIdx.x + u * kSTh;
        if (e < n) {
            out[atomicAdd(&cur[((uint32_t)x[u] - r.lo) >> s], 1u)] = Placed{x[u], (uint32_t)e, 0};
        }
    }
}

// Ranks of Q entries per lane (e0 + 64 q + lane) among the bucket's m keys in
// LDS: how many are smaller.  Keys are read 16 bytes at a time, two reads
// ahead; past the last one they are the largest value.
typedef uint32_t u4_t __attribute__((ext_vector_type(4), may_alias));
typedef uint64_t l2_t __attribute__((ext_vector_type(2), may_alias));
template <int Q, typename KEY>
__device__ __forceinline__ void ranks(const KEY* key, int m, int e0, int lane, int (&rank)[Q])
{
    using V = std::conditional_t<sizeof(KEY) == 4, u4_t, l2_t>;
    constexpr int N = 16 / sizeof(KEY);
    const V* const kv = reinterpret_cast<const V*>(key);
    KEY k[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int e = e0 + 64 * q + lane;
        k[q] = e < m ? key[e] : 0;
        rank[q] = 0;
    }
    V a = kv[0], b = kv[1];
    const int n = (m + 2 * N - 1) / (2 * N);
    for (int j = 0; j < n; ++j) {
        const V a1 = kv[2 * j + 2], b1 = kv[2 * j + 3];     // up to 32 bytes past the padding
#pragma unroll
        for (int v = 0; v < N; ++v)
#pragma unroll
            for (int q = 0; q < Q; ++q) rank[q] += (a[v] < k[q] ? 1 : 0) + (b[v] < k[q] ? 1 : 0);
        a = a1;
        b = b1;
    }
}

// LDS accesses of the wave's other lanes are done (its block's other waves
// have buckets of their own).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per bucket: an entry's place is the number of entries with a
// smaller (word, place in the input).  Words are compared alone first (half
// the work of the pair); where two are equal, they share a place and leave
// another without an entry, and the pairs are compared.  A bucket that does
// not fit the LDS (an input crowded into few words) is ordered by the wave in
// global memory: a bitonic network over the pairs, the entries past the end
// taken as the largest.
constexpr int kBucketWaves = 4;
__global__ __launch_bounds__(64 * kBucketWaves) void k_sort_buckets(uint64_t* __restrict__ cand, int bins,
                                                                    const uint32_t* __restrict__ start,
                                                                    Placed* __restrict__ placed)
{
    // a wave's keys (words, or pairs), padded with largest ones, and for words
    // the flags of the places taken
    constexpr int kPad = 8;
    __shared__ __align__(16) uint64_t keys[kBucketWaves * (kBucket + kPad)];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // the fullest buckets are neighbours (plane 1 of a row, at a fixed
    // distance from row to row): an odd stride over the power of two spreads
    // them over blocks, XCDs and compute units (305 K entries: 29.1 us with
    // neighbouring buckets in neighbouring blocks, 26.2 us so)
    const int b = (int)((blockIdx.x * kBucketWaves + wave) * 181u) & (bins - 1);
    if (b >= bins) return;
    const uint32_t first = start[b];
    const int m = __builtin_amdgcn_readfirstlane((int)(start[b + 1] - first));
    if (m == 0) return;
    uint64_t* const key = keys + wave * (kBucket + kPad);
    uint64_t* const out = cand + first;
    Placed* const in = placed + first;
    if (m <= kBucket) {
        uint32_t* const w = reinterpret_cast<uint32_t*>(key);
        uint32_t* const taken = w + kBucket + kPad;
        for (int e = lane; e < m; e += 64) {
            w[e] = (uint32_t)in[e].e;
            taken[e] = 0;
        }
        if (lane < kPad) w[m + lane] = ~0u;
        wave_sync();
        auto by_word = [&](auto qc) __attribute__((always_inline)) {
            constexpr int Q = decltype(qc)::value;
            for (int e0 = 0; e0 < m; e0 += 64 * Q) {
                int rank[Q];
                ranks<Q, uint32_t>(w, m, e0, lane, rank);
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int e = e0 + 64 * q + lane;
                    if (e < m) {
                        taken[rank[q]] = 1;
                        out[rank[q]] = in[e].e;
                    }
                }
            }
        };
        if (m <= 64) by_word(std::integral_constant<int, 1>{});
        else if (m <= 128) by_word(std::integral_constant<int, 2>{});
        else by_word(std::integral_constant<int, 4>{});
        wave_sync();
        bool clash = false;
        for (int e = lane; e < m; e += 64) clash |= taken[e] == 0;
        if (!__builtin_amdgcn_ballot_w64(clash)) return;
        wave_sync();
        for (int e = lane; e < m; e += 64) key[e] = ((uint64_t)(uint32_t)in[e].e << 32) | in[e].i;
        if (lane < kPad) key[m + lane] = ~0ull;
        wave_sync();
        for (int e0 = 0; e0 < m; e0 += 64) {
            int rank[1];
            ranks<1, uint64_t>(key, m, e0, lane, rank);
            if (e0 + lane < m) out[rank[0]] = in[e0 + lane].e;
        }
        return;
    }
    int p2 = 1;
    while (p2 < m) p2 <<= 1;
    for (int w = 2; w <= p2; w <<= 1) {
        for (int d = w >> 1; d > 0; d >>= 1) {
            for (int t = lane; t < p2 / 2; t += 64) {
                // the first step of a merge compares mirrored places, so that
                // every run is ascending and the missing entries stay last
                const int i = (t / d) * 2 * d + t % d;
                const int j = d == w >> 1 ? (i / w) * w + (w - 1 - i % w) : i + d;
                if (j < m) {
                    const uint64_t ei = in[i].e, ej = in[j].e;
                    const uint32_t pi = in[i].i, pj = in[j].i;
                    const uint64_t ki = ((uint64_t)(uint32_t)ei << 32) | pi, kj = ((uint64_t)(uint32_t)ej << 32) | pj;
                    if (ki > kj) {
                        in[i].e = ej;
                        in[i].i = pj;
                        in[j].e = ei;
                        in[j].i = pi;
                    }
                }
            }
            __threadfence_block();
            wave_sync();
        }
    }
    for (int e = lane; e < m; e += 64) out[e] = in[e].e;
}

struct SortLayout {
    size_t placed, parts, ph, sum, start, total;
};

SortLayout own_layout(int64_t n)
{
    SortLayout L;
    const int G = sort_blocks(n), bins = sort_bins(n);
    L.placed = 0;
    L.parts = L.placed + align_up((size_t)n * sizeof(Placed));
    L.ph = L.parts + align_up((size_t)G * sizeof(Range));
    L.sum = L.ph + align_up((size_t)G * bins * 4);
    L.start = L.sum + align_up((size_t)bins * 4);
    L.total = L.start + align_up((size_t)(bins + 1) * 4);
    return L;
}

}  // namespace

// Never less than for a shorter list (a caller may size its scratch for the
// longest list it will sort).
hipError_t sort_workspace(int64_t n, size_t* bytes)
{
    const size_t own = own_layout(n < kSortMax ? n : kSortMax).total;
    if (n <= kSortMax) {
        int dev = 0;
        const hipError_t e = hipGetDevice(&dev);
        *bytes = own;
        return e;
    }
    size_t temp = 0;
    rocprim::double_buffer<uint64_t> kb(nullptr, nullptr);
    hipError_t e = rocprim::radix_sort_keys(nullptr, temp, kb, (size_t)n, 0, 32);
    const size_t lib = align_up((size_t)n * 8) + temp;
    *bytes = lib > own ? lib : own;
    return e;
}

hipError_t sort_candidates(uint64_t* cand, int64_t n, void* work, hipStream_t s)
{
    if (n <= 1) return hipSuccess;
    if (n <= kSortMax) {
        const SortLayout L = own_layout(n);
        char* w = static_cast<char*>(work);
        Placed* placed = reinterpret_cast<Placed*>(w + L.placed);
        Range* parts = reinterpret_cast<Range*>(w + L.parts);
        uint32_t* ph = reinterpret_cast<uint32_t*>(w + L.ph);
        uint32_t* sum = reinterpret_cast<uint32_t*>(w + L.sum);
        uint32_t* start = reinterpret_cast<uint32_t*>(w + L.start);
        const int bins = sort_bins(n);
        if (n <= kSortOne) {
            hipLaunchKernelGGL(k_sort_one, dim3(1), dim3(kSTh), 0, s, cand, (int)n, bins, start, placed);
        } else {
            const int G = sort_blocks(n);
            hipLaunchKernelGGL(k_sort_range, dim3(G), dim3(kSTh), 0, s, cand, n, parts);
            hipLaunchKernelGGL(k_sort_hist, dim3(G), dim3(kSTh), 0, s, cand, n, bins, parts, ph);
            hipLaunchKernelGGL(k_sort_scan, dim3((bins + kScanTh - 1) / kScanTh), dim3(kScanTh), 0, s, ph, G, bins, sum);
            hipLaunchKernelGGL(k_sort_scatter, dim3(G), dim3(kSTh), 0, s, cand, n, bins, parts, ph, sum, start, placed);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_sort_buckets, dim3((unsigned)((bins + kBucketWaves - 1) / kBucketWaves)),
                           dim3(64 * kBucketWaves), 0, s, cand, bins, start, placed);
        return hipGetLastError();
    }
    uint64_t* alt = static_cast<uint64_t*>(work);
    void* temp = static_cast<char*>(work) + align_up((size_t)n * 8);
    size_t temp_bytes = 0;
    rocprim::double_buffer<uint64_t> kb(cand, alt);
    hipError_t e = rocprim::radix_sort_keys(nullptr, temp_bytes, kb, (size_t)n, 0, 32, s);
    if (e != hipSuccess) return e;
    e = rocprim::radix_sort_keys(temp, temp_bytes, kb, (size_t)n, 0, 32, s);
    if (e != hipSuccess) return e;
    if (kb.current() != cand)
        e = hipMemcpyAsync(cand, kb.current(), (size_t)n * 8, hipMemcpyDeviceToDevice, s);
    return e;
}

}  // namespace hsk
