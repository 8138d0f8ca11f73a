// Canonical order of a candidate list: ascending CL1 word (row, then plane,
// then bin), i.e. a stable sort of the 8-byte entries on their low 32 bits
// (the power in the high half travels with its word).
//
// A block sorts a list of up to 2048 entries (k_sort_one).  Longer ones, up to
// kSortMax, are parted into buckets first, and a block sorts each:
//   1. k_sort_hist     splitters (every kOver-th of a sorted sample) and the
//                      bucket counts per block;
//   2. k_sort_scatter  entries, each with its place in the input, to their
//                      buckets;
//   3. k_sort_buckets  one block per bucket.
// One block takes the place of 1 and 2 up to 16384 entries (k_sort_part).
//
// Splitters and entries are compared as (word, place in the input), which are
// all different, and the samples are taken at scattered places of the list: a
// bucket holds kOver gaps of the sample, whatever the words are (candidates
// crowd in plane 1, in the low bins, in a row with interference; of buckets of
// equal width a few would hold the list).  Inside a block, entries are ranked
// among those of the same bin of 2048 or 4096 (equal width); where the words
// are too crowded for that, or repeat, they are ordered eight bits at a time.
//
// What bounds it: latency, and scattered stores of a few MB in the L2.  Times:
// see sort_candidates.  Longer lists go to rocPRIM, which large passes suit.
#include <hip/hip_runtime.h>

#include <rocprim/device/device_radix_sort.hpp>

#include <type_traits>

#include "hs_internal.h"

namespace hsk {

namespace {

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int64_t kSortMax = (int64_t)1 << 20;
constexpr int kSTh = 1024;              // threads of the passes over the list, and of one sort
constexpr int kBTh = 512;               // threads that sort a bucket
constexpr int kBMax = 16;               // entries of a thread in a sort, at most
constexpr int64_t kSortOne = 2 * kSTh;
constexpr int64_t kSortPart = kBMax * kSTh;
constexpr int kBucket = kBTh * kBMax;   // entries of a bucket ordered in LDS
constexpr int kSortBlocks = 128;
constexpr int kSU = 4;                  // loads in flight per thread
constexpr int kBinsMax = 1024;
constexpr int kPartBins = 64;           // buckets of k_sort_part
constexpr int kOver = 4;                // samples per bucket
constexpr int kCrowd = 64;              // entries of a bin ranked one by one, at most
constexpr int kRadix = 256;
typedef uint64_t u64_alias __attribute__((may_alias));

int sort_blocks(int64_t n)
{
    const int64_t b = (n + (int64_t)kSTh * kSU - 1) / ((int64_t)kSTh * kSU);
    return (int)(b < 1 ? 1 : (b > kSortBlocks ? kSortBlocks : b));
}

// Buckets of a list: at most 512 entries in the mean (one a thread), or 1024
// above 2^18 entries (the counts of more buckets cost more than they save).
// The sum of kOver = 4 gaps of a random sample exceeds eight times its mean
// (kBucket, where the mean is 1024) with a probability below 1e-10.
int sort_bins(int64_t n)
{
    int b = kPartBins;
    while ((b < 512 && (int64_t)b * 512 < n) || (b < kBinsMax && (int64_t)b * 1024 < n)) b *= 2;
    return b;
}
static_assert(kSortMax <= (int64_t)kBinsMax * kBucket / 8, "eight times the mean of a bucket");
static_assert(kBinsMax * kOver <= kSTh * 4, "samples of k_sort_hist");

// LDS accesses of the wave's other lanes are done.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of a sort by NT threads of K entries each.
template <int NT, int K>
struct SortLds {
    uint64_t x[NT * K];
    union alignas(16) {
        uint16_t hist[(NT / 64) * kRadix];  // per wave and digit
        uint32_t bin[4 * NT];
    };
    uint16_t base[kRadix];
    uint32_t part[2 * (NT / 64)];
};

// Place of a thread's entry q: consecutive in a wave, waves in order.
template <int K>
__device__ __forceinline__ int place_of(int q)
{
    return (int)(threadIdx.x >> 6) * (64 * K) + 64 * q + (int)(threadIdx.x & 63);
}

// Smallest and largest word of the m entries; every thread gets them.
template <int NT, int K>
__device__ __forceinline__ void word_range(const uint64_t (&x)[K], int m, uint32_t* part, uint32_t& lo, uint32_t& hi)
{
    lo = ~0u;
    hi = 0;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (place_of<K>(q) < m) {
            const uint32_t w = (uint32_t)x[q];
            lo = w < lo ? w : lo;
            hi = w > hi ? w : hi;
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t l = (uint32_t)__shfl_xor((int)lo, d, 64), h = (uint32_t)__shfl_xor((int)hi, d, 64);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    constexpr int W = NT / 64;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6] = lo;
        part[W + (threadIdx.x >> 6)] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) {
        lo = part[w] < lo ? part[w] : lo;
        hi = part[W + w] > hi ? part[W + w] : hi;
    }
}

// Stable order of the m entries of the block by their low words lo..hi, eight
// bits at a time from the lowest.  Per digit: a wave ranks its entries, 64 at
// a time, by ballots of the digit's bits over its own counters; the counters
// are summed over digits, then waves; the entries move through LDS.  Places
// from m on hold nothing.  Entries are in x and, where there was a digit to
// sort by, in s.x.
template <int NT, int K>
__device__ __forceinline__ void by_words(uint64_t (&x)[K], int m, uint32_t lo, uint32_t hi, SortLds<NT, K>& s)
{
    constexpr int W = NT / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bits = hi == lo ? 0 : 32 - __builtin_clz(hi - lo);
    const int passes = (bits + 7) / 8;
    const int width = passes ? (bits + passes - 1) / passes : 0;
    uint16_t* const h = s.hist + wave * kRadix;
#pragma unroll 1
    for (int p = 0; p < passes; ++p) {
        const int shift = p * width;
        reinterpret_cast<u64_alias*>(h)[lane] = 0;
        wave_sync();
        uint32_t at[K];                 // digit, and place among the wave's of that digit
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const bool in = place_of<K>(q) < m;
            const uint32_t d = in ? (((uint32_t)x[q] - lo) >> shift) & ((1u << width) - 1u) : 0u;
            uint64_t same = __builtin_amdgcn_ballot_w64(in);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool set = (d >> b) & 1u;
                const uint64_t v = __builtin_amdgcn_ballot_w64(set);
                same &= set ? v : ~v;
            }
            const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0));
            const uint32_t old = h[d];
            wave_sync();
            if (in && before == 0) h[d] = (uint16_t)(old + __builtin_popcountll(same));
            wave_sync();
            at[q] = (d << 16) | (old + before);
        }
        __syncthreads();
        // thread d: the counters of digit d
        uint32_t sum = 0, inc = 0;
        if (threadIdx.x < kRadix) {
            uint32_t v[W];
#pragma unroll
            for (int w = 0; w < W; ++w) v[w] = s.hist[w * kRadix + threadIdx.x];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                s.hist[w * kRadix + threadIdx.x] = (uint16_t)sum;
                sum += v[w];
            }
            inc = sum;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = (uint32_t)__shfl_up((int)inc, d, 64);
                if (lane >= d) inc += o;
            }
            if (lane == 63) s.part[wave] = inc;
        }
        __syncthreads();
        if (threadIdx.x < kRadix) {
            for (int w = 0; w < wave; ++w) inc += s.part[w];
            s.base[threadIdx.x] = (uint16_t)(inc - sum);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const uint32_t d = at[q] >> 16;
            if (place_of<K>(q) < m) s.x[(uint32_t)s.base[d] + h[d] + (at[q] & 0xffffu)] = x[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < K; ++q)
            if (place_of<K>(q) < m) x[q] = s.x[place_of<K>(q)];
    }
}
static_assert(4 * kSTh < 65536 && kBucket < 65536, "places and counters of 16 bits");

// Places of the m entries in the order of their low words lo..hi (of (low, high
// word) if WHOLE: all different then): they are parted into 4 NT bins of equal
// width in LDS and ranked inside their bin.  False where a bin holds more than
// kCrowd entries, or two words are equal; x is left as it was.
template <int NT, int K, bool WHOLE>
__device__ __forceinline__ bool by_bins(const uint64_t (&x)[K], int m, uint32_t lo, uint32_t hi, SortLds<NT, K>& s,
                                        int (&to)[K])
{
    typedef uint32_t four __attribute__((ext_vector_type(4), may_alias));
    constexpr int B = 4 * NT;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bits = hi == lo ? 0 : 32 - __builtin_clz(hi - lo), have = 31 - __builtin_clz((uint32_t)B);
    const int shift = bits > have ? bits - have : 0;
    four* const mine = reinterpret_cast<four*>(s.bin) + threadIdx.x;
    *mine = four{0, 0, 0, 0};
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q)
        to[q] = place_of<K>(q) < m ? (int)atomicAdd(&s.bin[((uint32_t)x[q] - lo) >> shift], 1u) : 0;
    __syncthreads();
    const four c = *mine;
    uint32_t inc = c.x + c.y + c.z + c.w;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) s.part[wave] = inc;
    if (__syncthreads_or(c.x > kCrowd || c.y > kCrowd || c.z > kCrowd || c.w > kCrowd)) return false;
    for (int w = 0; w < wave; ++w) inc += s.part[w];
    *mine = four{inc - c.w - c.z - c.y - c.x, inc - c.w - c.z - c.y, inc - c.w - c.z, inc - c.w};
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q)
        if (place_of<K>(q) < m) s.x[s.bin[((uint32_t)x[q] - lo) >> shift] + to[q]] = x[q];
    __syncthreads();
    bool equal = false;
#pragma unroll
    for (int q = 0; q < K; ++q) {
        if (place_of<K>(q) < m) {
            const int b = (int)(((uint32_t)x[q] - lo) >> shift);
            const int first = (int)s.bin[b], last = b + 1 < B ? (int)s.bin[b + 1] : m;
            const uint64_t key = (x[q] << 32) | (x[q] >> 32);
            int less = 0, same = 0;
            for (int e = first; e < last; ++e) {
                const uint64_t y = s.x[e];
                if constexpr (WHOLE) {
                    less += ((y << 32) | (y >> 32)) < key ? 1 : 0;
                } else {
                    less += (uint32_t)y < (uint32_t)x[q] ? 1 : 0;
                    same += (uint32_t)y == (uint32_t)x[q] ? 1 : 0;
                }
            }
            to[q] = first + less;
            equal |= !WHOLE && same > 1;
        }
    }
    return !__syncthreads_or(equal);
}

// A whole list in one block (n <= K kSTh).
template <int K>
__global__ __launch_bounds__(kSTh) void k_sort_one(uint64_t* __restrict__ cand, int n)
{
    extern __shared__ __align__(16) unsigned char smem[];
    SortLds<kSTh, K>& s = *reinterpret_cast<SortLds<kSTh, K>*>(smem);
    uint64_t x[K];
#pragma unroll
    for (int q = 0; q < K; ++q) x[q] = place_of<K>(q) < n ? cand[place_of<K>(q)] : 0;
    uint32_t lo, hi;
    word_range<kSTh, K>(x, n, s.part, lo, hi);
    int to[K];
    if (!by_bins<kSTh, K, false>(x, n, lo, hi, s, to)) {
        by_words<kSTh, K>(x, n, lo, hi, s);
#pragma unroll
        for (int q = 0; q < K; ++q) to[q] = place_of<K>(q);
    }
#pragma unroll
    for (int q = 0; q < K; ++q)
        if (place_of<K>(q) < n) cand[to[q]] = x[q];
}

// Place of sample i of S: the list is cut into S runs of equal length, and one
// entry of each is taken, at a place of the run that looks random.
__device__ __forceinline__ int64_t sample_place(uint32_t i, int64_t n, uint32_t S)
{
    const int64_t a = (int64_t)i * n / S, b = (int64_t)(i + 1) * n / S;
    uint32_t h = (i + 1) * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    h ^= h >> 13;
    return a + (int64_t)(((uint64_t)h * (uint64_t)(b - a)) >> 32);
}

// The splitters (word, place) of `bins` buckets: split[b] is the smallest that
// belongs to bucket b.  Samples are taken in the order of their places, so the
// stable sort leaves equal words in that order.
template <int K>
__device__ __forceinline__ void splitters(const uint64_t* __restrict__ cand, int64_t n, int bins, uint64_t* split,
                                          SortLds<kSTh, K>& s)
{
    const int S = bins * kOver;
    uint64_t x[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const int i = place_of<K>(q);
        const int64_t at = sample_place((uint32_t)(i < S ? i : S - 1), n, (uint32_t)S);
        x[q] = ((uint64_t)at << 32) | (uint32_t)cand[at];
    }
    uint32_t lo, hi;
    word_range<kSTh, K>(x, S, s.part, lo, hi);
    int to[K];
    if (!by_bins<kSTh, K, true>(x, S, lo, hi, s, to)) {
        by_words<kSTh, K>(x, S, lo, hi, s);
#pragma unroll
        for (int q = 0; q < K; ++q) to[q] = place_of<K>(q);
    }
#pragma unroll
    for (int q = 0; q < K; ++q)
        if (place_of<K>(q) < S && to[q] % kOver == 0) split[to[q] / kOver] = to[q] == 0 ? 0 : (x[q] << 32) | (x[q] >> 32);
}

__device__ __forceinline__ void chunk(int64_t n, int64_t& e0, int64_t& e1)
{
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    e0 = (int64_t)blockIdx.x * per;
    e1 = e0 + per < n ? e0 + per : n;
    if (e0 > n) e0 = n;
}

// f(entry, place, bucket) for the block's entries, kSU loads and searches in
// flight per thread.
template <typename F>
__device__ __forceinline__ void each(const uint64_t* __restrict__ a, int64_t n, const uint64_t* sp, int bins, F f)
{
    int64_t e0, e1;
    chunk(n, e0, e1);
    for (int64_t b = e0 + threadIdx.x; b < e1; b += (int64_t)kSU * kSTh) {
        uint64_t x[kSU], key[kSU];
        int at[kSU];
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
            const int64_t e = b + (int64_t)u * kSTh;
            x[u] = a[e < e1 ? e : e1 - 1];
        }
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
            key[u] = (x[u] << 32) | (uint32_t)(b + (int64_t)u * kSTh);
            at[u] = 0;
        }
        // the last splitter that is not larger (bins is a power of two)
        for (int h = bins >> 1; h > 0; h >>= 1) {
#pragma unroll
            for (int u = 0; u < kSU; ++u) at[u] += sp[at[u] + h] <= key[u] ? h : 0;
        }
#pragma unroll
        for (int u = 0; u < kSU; ++u)
            if (b + (int64_t)u * kSTh < e1) f(x[u], (uint32_t)key[u], at[u]);
    }
}

// Every block finds the splitters for itself (the first hands them on): a pass
// of its own would take a launch.
template <int K>
__global__ __launch_bounds__(kSTh) void k_sort_hist(const uint64_t* __restrict__ cand, int64_t n, int bins,
                                                    uint64_t* __restrict__ split, uint32_t* __restrict__ ph)
{
    extern __shared__ __align__(16) unsigned char smem[];
    SortLds<kSTh, K>& s = *reinterpret_cast<SortLds<kSTh, K>*>(smem);
    uint64_t* const sp = reinterpret_cast<uint64_t*>(smem + sizeof(s));
    uint32_t* const hist = reinterpret_cast<uint32_t*>(sp + bins);
    for (int i = threadIdx.x; i < bins; i += kSTh) hist[i] = 0;
    splitters<K>(cand, n, bins, sp, s);
    __syncthreads();
    each(cand, n, sp, bins, [&](uint64_t, uint32_t, int b) { atomicAdd(&hist[b], 1u); });
    __syncthreads();
    for (int i = threadIdx.x; i < bins; i += kSTh) {
        ph[(int64_t)blockIdx.x * bins + i] = hist[i];
        if (blockIdx.x == 0) split[i] = sp[i];
    }
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
    return before + inc - v;
}

// An entry with its place in the input.
struct alignas(16) Placed {
    uint64_t e;
    uint32_t i, pad;
};

// Each block sums the counts itself (at most 512 KB from the L2), which a pass
// of its own would take a launch for.
__global__ __launch_bounds__(kSTh) void k_sort_scatter(const uint64_t* __restrict__ cand, int64_t n, int bins,
                                                       const uint64_t* __restrict__ split,
                                                       const uint32_t* __restrict__ ph, uint32_t* __restrict__ start,
                                                       Placed* __restrict__ out)
{
    __shared__ uint64_t sp[kBinsMax];
    __shared__ uint32_t cur[kBinsMax], total[kBinsMax];
    const int t = threadIdx.x, G = gridDim.x, me = blockIdx.x;
    if (t < bins) {
        sp[t] = split[t];
        cur[t] = 0;
        total[t] = 0;
    }
    __syncthreads();
    // kSTh / bins threads per bucket, each a run of the blocks
    {
        const int b = t & (bins - 1), runs = kSTh / bins, r = t / bins;
        const int g0 = r * G / runs, g1 = (r + 1) * G / runs;
        uint32_t all = 0, mine = 0;
        for (int g = g0; g < g1; g += 16) {
            uint32_t v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = ph[(int64_t)(g + q < g1 ? g + q : g1 - 1) * bins + b];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                all += g + q < g1 ? v[q] : 0u;
                mine += g + q < g1 && g + q < me ? v[q] : 0u;
            }
        }
        if (all) atomicAdd(&total[b], all);
        if (mine) atomicAdd(&cur[b], mine);
    }
    __syncthreads();
    const uint32_t tot = t < bins ? total[t] : 0u;
    const uint32_t at = block_exclusive(tot);
    if (t < bins) {
        cur[t] += at;
        if (me == 0) {
            start[t] = at;
            if (t == bins - 1) start[bins] = at + tot;
        }
    }
    __syncthreads();
    each(cand, n, sp, bins, [&](uint64_t x, uint32_t i, int b) { out[atomicAdd(&cur[b], 1u)] = Placed{x, i, 0}; });
}

// The passes before the buckets for a list of up to K kSTh entries, in one
// block (16 384 entries 24 us so, 26 in three launches): buckets of equal width
// where none of them holds much more than its share (which saves sorting
// samples and searching), else splitters.
template <int K>
__global__ __launch_bounds__(kSTh) void k_sort_part(const uint64_t* __restrict__ cand, int n,
                                                    uint32_t* __restrict__ start, Placed* __restrict__ out)
{
    __shared__ uint64_t sp[kPartBins];
    __shared__ uint32_t cur[kPartBins];
    __shared__ SortLds<kSTh, 1> s;
    const int t = threadIdx.x;
    uint64_t x[K];
#pragma unroll
    for (int q = 0; q < K; ++q) x[q] = place_of<K>(q) < n ? cand[place_of<K>(q)] : 0;
    if (t < kPartBins) cur[t] = 0;
    uint32_t lo, hi;
    word_range<kSTh, K>(x, n, s.part, lo, hi);
    constexpr int have = 31 - __builtin_clz((uint32_t)kPartBins);
    const int bits = hi == lo ? 0 : 32 - __builtin_clz(hi - lo), shift = bits > have ? bits - have : 0;
    uint32_t at[K];                     // bucket, and place among its entries
    auto count = [&](int q, uint32_t b) __attribute__((always_inline)) {
        at[q] = place_of<K>(q) < n ? (b << 16) | atomicAdd(&cur[b], 1u) : 0u;
    };
    // the first entry of every thread tells most crowded lists
    count(0, ((uint32_t)x[0] - lo) >> shift);
    __syncthreads();
    bool crowded = __syncthreads_or(t < kPartBins && cur[t] > (1u << 20) / (uint32_t)n);
    if (!crowded) {
#pragma unroll
        for (int q = 1; q < K; ++q) count(q, ((uint32_t)x[q] - lo) >> shift);
        __syncthreads();
        crowded = __syncthreads_or(t < kPartBins && cur[t] > 2 * kBTh);
    }
    if (crowded) {
        splitters<1>(cand, n, kPartBins, sp, s);
        if (t < kPartBins) cur[t] = 0;
        __syncthreads();
        int b[K];
#pragma unroll
        for (int q = 0; q < K; ++q) b[q] = 0;
#pragma unroll
        for (int h = kPartBins / 2; h > 0; h >>= 1)
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const uint64_t key = (x[q] << 32) | (uint32_t)place_of<K>(q);
                b[q] += sp[b[q] + h] <= key ? h : 0;
            }
#pragma unroll
        for (int q = 0; q < K; ++q) count(q, (uint32_t)b[q]);
        __syncthreads();
    }
    const uint32_t mine = t < kPartBins ? cur[t] : 0u;
    const uint32_t first = block_exclusive(mine);
    if (t < kPartBins) {
        cur[t] = first;
        start[t] = first;
        if (t == kPartBins - 1) start[kPartBins] = first + mine;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q)
        if (place_of<K>(q) < n)
            out[cur[at[q] >> 16] + (at[q] & 0xffffu)] = Placed{x[q], (uint32_t)place_of<K>(q), 0};
}
static_assert(kSortPart < 65536 && kPartBins * kOver <= kSTh, "places of 16 bits, one sample per thread");

// One block per bucket (of half as many threads for the small buckets of a
// short list).  Entries come in no order, so equal words (which lists
// of several FOPs have) are told apart by their places: where two meet, the
// entries are put in the order of their places first, and sorted again.
template <int NT, int K>
__device__ __forceinline__ void sort_bucket(uint64_t* __restrict__ out, const Placed* __restrict__ in, int m,
                                            unsigned char* smem)
{
    SortLds<NT, K>& s = *reinterpret_cast<SortLds<NT, K>*>(smem);
    uint64_t x[K];
    uint32_t lo, hi;
#pragma unroll
    for (int q = 0; q < K; ++q) x[q] = place_of<K>(q) < m ? in[place_of<K>(q)].e : 0;
    word_range<NT, K>(x, m, s.part, lo, hi);
    if constexpr (K < kBMax) {          // (kBMax: registers)
        int to[K];
        if (by_bins<NT, K, false>(x, m, lo, hi, s, to)) {
#pragma unroll
            for (int q = 0; q < K; ++q)
                if (place_of<K>(q) < m) out[to[q]] = x[q];
            return;
        }
    }
    by_words<NT, K>(x, m, lo, hi, s);
    bool equal = lo == hi && m > 1;
    if (lo != hi) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int e = place_of<K>(q) + 1;
            equal |= e < m && (uint32_t)s.x[e] == (uint32_t)x[q];
        }
    }
    if (__syncthreads_or(equal)) {
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int e = place_of<K>(q);
            x[q] = ((uint64_t)(uint32_t)e << 32) | (e < m ? in[e].i : 0u);
        }
        uint32_t p0, p1;
        word_range<NT, K>(x, m, s.part, p0, p1);
        by_words<NT, K>(x, m, p0, p1, s);
#pragma unroll
        for (int q = 0; q < K; ++q)
            if (place_of<K>(q) < m) x[q] = in[x[q] >> 32].e;
        __syncthreads();
        by_words<NT, K>(x, m, lo, hi, s);
    }
#pragma unroll
    for (int q = 0; q < K; ++q)
        if (place_of<K>(q) < m) out[place_of<K>(q)] = x[q];
}

// A small bucket (m <= NT): each entry's word is compared with all others, which no
// crowd of words slows down.  False, with nothing written, where two are equal.
template <int NT>
__device__ __forceinline__ bool rank_all(uint64_t* __restrict__ out, const Placed* __restrict__ in, int m,
                                         unsigned char* smem)
{
    typedef uint32_t four __attribute__((ext_vector_type(4), may_alias));
    uint32_t* const word = reinterpret_cast<uint32_t*>(smem);
    uint32_t* const given = word + NT;
    const int t = threadIdx.x;
    const uint64_t x = in[t < m ? t : 0].e;
    const uint32_t w = (uint32_t)x;
    word[t] = t < m ? w : ~0u;          // past the end: below no word
    given[t] = 0;
    __syncthreads();
    int rank = 0;
    if (t < m) {
        for (int e = 0; e < m; e += 4) {
            const four y = *reinterpret_cast<const four*>(word + e);
            rank += (y.x < w ? 1 : 0) + (y.y < w ? 1 : 0) + (y.z < w ? 1 : 0) + (y.w < w ? 1 : 0);
        }
    }
    // equal words get the same rank
    if (__syncthreads_or(t < m && atomicAdd(&given[rank], 1u) > 0)) return false;
    if (t < m) out[rank] = x;
    return true;
}

template <int NT>
__global__ __launch_bounds__(NT, 4) void k_sort_buckets(uint64_t* __restrict__ cand,
                                                          const uint32_t* __restrict__ start,
                                                          Placed* __restrict__ placed)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t first = start[blockIdx.x];
    const int m = __builtin_amdgcn_readfirstlane((int)(start[blockIdx.x + 1] - first));
    if (m == 0) return;
    uint64_t* const out = cand + first;
    Placed* const in = placed + first;
    // the 64 buckets of a short list: 2500 entries 15.5 -> 14.7 us, 9000 at log-
    // uniform bins 22 -> 20, 9000 in one row 31 -> 29 (buckets of up to 512 so:
    // 16 384 entries 24 -> 27)
    if (NT == kBTh / 2 && m <= NT && rank_all<NT>(out, in, m, smem)) return;
    if (m <= NT) return sort_bucket<NT, 1>(out, in, m, smem);
    if (m <= 2 * NT) return sort_bucket<NT, 2>(out, in, m, smem);
    if (m <= 4 * NT) return sort_bucket<NT, 4>(out, in, m, smem);
    if (m <= 8 * NT) return sort_bucket<NT, 8>(out, in, m, smem);
    if (m <= kBMax * NT) return sort_bucket<NT, kBMax>(out, in, m, smem);
    // not by chance: a list made so that the samples miss most of it.  A
    // bitonic network over (word, place) in global memory, the entries past
    // the end taken as the largest.
    int p2 = 1;
    while (p2 < m) p2 <<= 1;
    for (int w = 2; w <= p2; w <<= 1) {
        for (int d = w >> 1; d > 0; d >>= 1) {
            for (int t = threadIdx.x; t < p2 / 2; t += NT) {
                // the first step of a merge compares mirrored places, so that
                // every run is ascending and the missing entries stay last
                const int i = (t / d) * 2 * d + t % d;
                const int j = d == w >> 1 ? (i / w) * w + (w - 1 - i % w) : i + d;
                if (j < m) {
                    const uint64_t ei = in[i].e, ej = in[j].e;
                    const uint32_t pi = in[i].i, pj = in[j].i;
                    const uint64_t ki = (ei << 32) | pi, kj = (ej << 32) | pj;
                    if (ki > kj) {
                        in[i].e = ej;
                        in[i].i = pj;
                        in[j].e = ei;
                        in[j].i = pi;
                    }
                }
            }
            __threadfence_block();
            __syncthreads();
        }
    }
    for (int e = threadIdx.x; e < m; e += NT) out[e] = in[e].e;
}

struct SortLayout {
    size_t placed, split, ph, start, total;
};

SortLayout own_layout(int64_t n)
{
    SortLayout L;
    const int G = sort_blocks(n), bins = sort_bins(n);
    L.placed = 0;
    L.split = L.placed + align_up((size_t)n * sizeof(Placed));
    L.ph = L.split + align_up((size_t)bins * 8);
    L.start = L.ph + align_up((size_t)G * bins * 4);
    L.total = L.start + align_up((size_t)(bins + 1) * 4);
    return L;
}

template <int K>
hipError_t launch_one(uint64_t* cand, int n, hipStream_t s)
{
    constexpr int lds = sizeof(SortLds<kSTh, K>);
    hipLaunchKernelGGL(k_sort_one<K>, dim3(1), dim3(kSTh), lds, s, cand, n);
    return hipGetLastError();
}

template <int K>
hipError_t launch_hist(const uint64_t* cand, int64_t n, int bins, uint64_t* split, uint32_t* ph, int G, hipStream_t s)
{
    const int lds = (int)sizeof(SortLds<kSTh, K>) + bins * 12;
    hipLaunchKernelGGL(k_sort_hist<K>, dim3(G), dim3(kSTh), lds, s, cand, n, bins, split, ph);
    return hipGetLastError();
}
static_assert(sizeof(SortLds<kSTh, 4>) + kBinsMax * 12 <= 65536 && sizeof(SortLds<kSTh, 4>) % 8 == 0,
              "LDS without asking for more");

template <int NT>
hipError_t launch_buckets(uint64_t* cand, const uint32_t* start, Placed* placed, int bins, hipStream_t s)
{
    constexpr int lds = sizeof(SortLds<NT, kBMax>);
    if (lds > 65536)
        (void)hipFuncSetAttribute((const void*)k_sort_buckets<NT>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    hipLaunchKernelGGL(k_sort_buckets<NT>, dim3(bins), dim3(NT), lds, s, cand, start, placed);
    return hipGetLastError();
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

// us a call on one MI355X, rocPRIM / buckets of equal width with a wave each /
// this: entries as a search of 85 x 2^21 finds them (plane 1 half of them), all
// in the lowest eighth of the bins, nine tenths in one row.
//     n        searched           low bins            one row
//     1 000     15 / 13 / 11       15 / 13 / 11        15 / 92 / 16
//     5 000     31 / 16 / 17       32 / 16 / 17        32 / 1040 / 31
//    16 384     34 / 27 / 24       35 / 26 / 26        35 / 2600 / 41
//    50 000     48 / 29 / 28       48 / 41 / 31        48 / 6000 / 35
//   305 000    124 / 60 / 44      125 / 580 / 57      122 / 12 700 / 50
//      2^20    188 / 225 / 81     188 / 3400 / 96     188 / 36 900 / 88
// Of the 38 us of kernels at 305 000 the counts take 14 (three of them the
// sample), the scatter 13, the buckets 10.
hipError_t sort_candidates(uint64_t* cand, int64_t n, void* work, hipStream_t s)
{
    if (n <= 1) return hipSuccess;
    if (n <= kSortOne) {
        if (n <= kSTh) return launch_one<1>(cand, (int)n, s);
        return launch_one<2>(cand, (int)n, s);
    }
    if (n <= kSortMax) {
        const SortLayout L = own_layout(n);
        char* w = static_cast<char*>(work);
        Placed* placed = reinterpret_cast<Placed*>(w + L.placed);
        uint64_t* split = reinterpret_cast<uint64_t*>(w + L.split);
        uint32_t* ph = reinterpret_cast<uint32_t*>(w + L.ph);
        uint32_t* start = reinterpret_cast<uint32_t*>(w + L.start);
        const int G = sort_blocks(n), bins = sort_bins(n), S = bins * kOver;
        hipError_t e = hipSuccess;
        if (n <= kSortPart) {
            if (n <= 4 * kSTh) hipLaunchKernelGGL(k_sort_part<4>, dim3(1), dim3(kSTh), 0, s, cand, (int)n, start, placed);
            else if (n <= 8 * kSTh) hipLaunchKernelGGL(k_sort_part<8>, dim3(1), dim3(kSTh), 0, s, cand, (int)n, start, placed);
            else hipLaunchKernelGGL(k_sort_part<kBMax>, dim3(1), dim3(kSTh), 0, s, cand, (int)n, start, placed);
            e = hipGetLastError();
        } else {
            e = S <= kSTh       ? launch_hist<1>(cand, n, bins, split, ph, G, s)
                : S <= 2 * kSTh ? launch_hist<2>(cand, n, bins, split, ph, G, s)
                                : launch_hist<4>(cand, n, bins, split, ph, G, s);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_sort_scatter, dim3(G), dim3(kSTh), 0, s, cand, n, bins, split, ph, start, placed);
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
        return n <= kSortPart ? launch_buckets<kBTh / 2>(cand, start, placed, bins, s)
                              : launch_buckets<kBTh>(cand, start, placed, bins, s);
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
