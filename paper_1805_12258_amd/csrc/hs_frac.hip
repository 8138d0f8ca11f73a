// Harmonic planes under the fractional mapping,
//     HPF_k(i, j) = sum_{m=1..k} FOP(floor(m i / k), floor(m j / k)),
// the FOP at the fractions m/k of each point (i = r - T/2 signed, floor
// division), terms added in the order m = 1..k in fp32 (each partial sum
// rounded, no contraction): the incoherent-sum reading of the harmonic sum
// of Sec. III.  Unlike Eq. 1-2 the planes are not cumulative: plane k reads
// k source points of its own, sum_k k = H (H + 1) / 2 of them per point.
//
// Chains.  m/K for m = 1..K holds every fraction of K, K/2, K/4, ... (while
// even), so one pass over the K sources of a row forms all those planes, and
// every k <= H/2 belongs to exactly one K in (H/2, H].  H = 8: 26 sources a
// point instead of 36, H = 16: 100 instead of 136.
//
// Layout of the work: a wave walks a few consecutive rows of one chain over a
// strip of 256 bins (four consecutive bins per lane).  Per source, a lane's
// bins lie in at most four consecutive elements (the source bin advances by
// m/K <= 1), which come with one vector load (element aligned, of just the
// elements that can be needed) and are picked per bin by the remainder of
// m j / K; source m changes its row in m of K rows only and is kept in
// registers otherwise.  Only the last strip of a ragged plane could read past
// it; it clamps each element.  The chains of some rows, then the rows of a
// strip, then strips follow one another on an XCD, so that the source rows of
// neighbours and of the chains (all read m = K) meet in its L2.
//
// What bounds it: the L1's access rate (13 accesses per unaligned vector load
// of a wave, which keeping the sources saves 44 % of) and, as much, the
// caches' traffic: 85 x 2^19, H = 8, fp32 fetches 1.37 GB (7.7 planes) in 207
// us.  One load per bin and term took 817 us (fp16, 2^18 bins: 504 us, now 84;
// H = 16 fp16 2^18: 1790 us, now 292; 127 x 2^20 at H = 4: 1176 us, now 198).
//
// Detection: the candidates of each (row, plane) are compacted with wave
// ballots into a per-wave LDS buffer and counted per plane in LDS; a full
// buffer is written out with one atomic that reserves its places, and the
// counters are added once per block of the resident grid.
#include <hip/hip_runtime.h>

#include "hs_rows.h"

namespace hsk {

namespace {

using rows::gptr_t;

constexpr int kFV = 4;                     // bins per lane
constexpr int kFBins = 64 * kFV;           // bins per strip
constexpr int kFCandCap = 320;             // per-wave LDS candidate buffer (>= kFBins)
// Waves of a block, and per SIMD: every block ends with an atomic per plane on
// the same few words (7-9 ns each), so few large blocks; the sources of chains
// above 8 need 128 registers.  85 x 2^19 fp32 at H = 8: 233 us with 4 waves,
// 207 with 8, 220 with 16 (one block less fits); 85 x 2^18 fp16 at H = 16: 379,
// 338 and 292.
constexpr int frac_waves(int G) { return G == 1 ? 8 : 16; }
constexpr int frac_occ(int G) { return G == 1 ? 6 : 4; }
constexpr int kFUnits = 3;                 // units of a wave, at least where there are rows for them
constexpr int kFRows = 16;                 // rows of a unit, at most

constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

// The remainders m j mod K of a lane's first bin j (a multiple of kFV) are
// multiples of this.
constexpr int rem_step(int m, int K) { return gcd_c(kFV * m, K); }

// Elements that a lane's kFV bins can reach from its first bin's source.
constexpr int span(int m, int K) { return (K - rem_step(m, K) + (kFV - 1) * m) / K + 1; }

// Bit sets over the sources m = 1..K of a row with e = i mod K (bit m - 1),
// for the source rows floor(m i / K):
//   first: the row of m is one further from that of m - 1 than floor(i / K);
//   next:  the row of m is another one than at i - 1.
constexpr uint32_t step_bits(int K, int e, bool next)
{
    uint32_t x = 0;
    for (int m = 1; m <= K; ++m)
        if (next ? e == 0 || m * e / K != m * (e - 1) / K : m * e / K != (m - 1) * e / K) x |= 1u << (m - 1);
    return x;
}

// word w of the sets: eight of 8 bits (K <= 8) or four of 16
constexpr uint64_t step_word(int K, int w, bool next)
{
    const int bits = K <= 8 ? 8 : 16, per = 64 / bits;
    uint64_t x = 0;
    for (int i = 0; i < per; ++i)
        if (per * w + i < K) x |= (uint64_t)step_bits(K, per * w + i, next) << (bits * i);
    return x;
}

template <int K, bool NEXT>
__device__ __forceinline__ uint32_t row_steps(int e)
{
    if constexpr (K <= 8) {
        constexpr uint64_t w0 = step_word(K, 0, NEXT);
        return (uint32_t)(w0 >> (8 * e));
    } else {
        constexpr uint64_t w0 = step_word(K, 0, NEXT), w1 = step_word(K, 1, NEXT), w2 = step_word(K, 2, NEXT),
                           w3 = step_word(K, 3, NEXT);
        const uint64_t w = e < 8 ? (e < 4 ? w0 : w1) : (e < 12 ? w2 : w3);
        return (uint32_t)(w >> (16 * (e & 3)));
    }
}

typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void store4(float* dst, const float* y)
{
    *reinterpret_cast<float4_a4*>(dst) = float4_a4{y[0], y[1], y[2], y[3]};
}

__device__ __forceinline__ uint32_t mul24(uint32_t x, uint32_t y) { return (x & 0xffffffu) * (y & 0xffffffu); }

// A wave's candidates: its buffer, and the block's counters.
struct Found {
    uint64_t* buf;
    uint32_t* cnt;    // [H], the block's
    int n;
};

__device__ __forceinline__ void put(const FracArgs& a, const Found& f, unsigned long long base, int lane)
{
    for (int e0 = 0; e0 < f.n; e0 += 64) {
        const int e = e0 + lane;
        if (e < f.n && (int64_t)(base + e) < a.cap) reinterpret_cast<uint64_t*>(a.out)[base + e] = f.buf[e];
    }
}

__device__ __forceinline__ void flush(const FracArgs& a, Found& f, int lane)
{
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&a.counts[a.H], (unsigned long long)f.n);
    put(a, f, (unsigned long long)rows::uni64((int64_t)base), lane);
    f.n = 0;
}

// Rows r0 <= r < r1 of the planes K, K/2, K/4, ... of a strip at j0.
template <typename TIn, int K, bool DETECT, bool EDGE>
__device__ __forceinline__ void chain(const FracArgs& a, Found& f, int j0, int r0, int r1, int lane)
{
    constexpr int EB = sizeof(TIn);
    constexpr int NP = __builtin_ctz(K) + 1;            // planes of the chain
    // opaque: the offsets of all chains are not formed ahead of the first
    const uint32_t jl = rows::opaque((uint32_t)j0 + (uint32_t)(kFV * lane));
    const int64_t ldb = a.ld * EB;
    const int T = rows::opaque_s(a.T);      // nor the offsets of the thresholds
    // m j = m K Q + m e with e < K: the first bin's source element is m Q +
    // floor(m e / K) (all of it full-rate 24-bit arithmetic: N <= 2^24, and
    // m e < K^2 <= 256, for which 65536 / K + 1 is an exact reciprocal)
    const uint32_t Q = jl / (uint32_t)K, e0 = jl - Q * (uint32_t)K;
    uint32_t q[K + 1], rem[K + 1];
    rows::static_for<1, K>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        const uint32_t me = mul24(e0, m), fl = mul24(me, 65536 / K + 1) >> 16;
        q[m] = (K == 1 ? jl : mul24(Q, m) + fl) * EB;
        rem[m] = me - mul24(fl, K);
    });
    // row c + floor(m i / K) of source m
    const int over = (a.c + K - 1) / K;                 // i + over K >= 0
    const int d0 = (int)((uint32_t)(r0 - a.c + over * K) / (uint32_t)K) - over;
    int e = r0 - a.c - d0 * K;
    gptr_t at[K + 1];
    {
        const int64_t step0 = d0 * ldb, step1 = step0 + ldb;
        const uint32_t up = row_steps<K, false>(e);
        gptr_t p = (gptr_t)(uintptr_t)a.fop + a.c * ldb;
        rows::static_for<1, K>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            p += up & (1u << (m - 1)) ? step1 : step0;
            at[m] = p;
        });
    }
    uint32_t raw[K + 1][4];
    uint32_t changed = (uint32_t)rows::opaque_s(-1);
#pragma unroll 1
    for (int row = r0; row < r1; ++row) {
        const int r = rows::opaque_s(row);
        const float* const tr = DETECT ? a.ta + r : nullptr;
        // the thresholds and the sources whose row is another one now, all
        // requested before the first is used
        float thr[NP];
        if constexpr (DETECT)
            rows::static_for<0, NP - 1>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                thr[t] = tr[(int64_t)((K >> t) - 1) * T];
            });
        rows::static_for<1, K>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int W = span(m, K);
            if (changed & (1u << (m - 1))) {
                const gptr_t p = rows::scalar(at[m]);
                if constexpr (EDGE) {
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        uint32_t o = rows::opaque(q[m]) + w * EB;
                        if (o > (uint32_t)(a.N - 1) * EB) o = (uint32_t)(a.N - 1) * EB;
                        uint32_t x[1];
                        rows::load_words<EB == 4 ? 1 : 0, EB>(p + o, x);
                        raw[m][w] = x[0];
                    }
                } else {
                    rows::load_words<EB == 4 ? W : (W == 1 ? 0 : (W + 1) / 2), EB>(p + rows::opaque(q[m]), raw[m]);
                }
            }
        });
        float acc[NP][kFV];
        rows::static_for<1, K>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int g = rem_step(m, K);
            constexpr int W = span(m, K);
            float x4[kFV];
#pragma unroll
            for (int w = 0; w < W; ++w)
                x4[w] = EDGE ? rows::decode<TIn>(&raw[m][w], 0) : rows::decode<TIn>(raw[m], w);
            // (compared once for all rows while the masks fit the scalar
            // registers)
            const uint32_t rm = K <= 8 ? rem[m] : rows::opaque(rem[m]);
#pragma unroll
            for (int v = 0; v < kFV; ++v) {
                const int lo = v * m / K;
                const int left = v * m % K;             // one more element where rem + left >= K
                float x = x4[lo];
                if (left >= g) x = rm >= (uint32_t)(K - left) ? x4[lo + 1] : x;
                rows::static_for<0, NP - 1>([&](auto tc) {
                    constexpr int t = decltype(tc)::value;
                    if constexpr (m % (1 << t) == 0) acc[t][v] = m == (1 << t) ? x : acc[t][v] + x;
                });
            }
        });
        rows::static_for<0, NP - 1>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            constexpr int k = K >> t;
            if constexpr (DETECT) {
                const float lim = thr[t] * a.scale;
                bool hit[kFV];
                bool anyl = false;
                if constexpr (EDGE) {
#pragma unroll
                    for (int v = 0; v < kFV; ++v) anyl |= jl + v < (uint32_t)a.N && acc[t][v] > lim;
                } else {
                    anyl = __builtin_fmaxf(__builtin_fmaxf(acc[t][0], acc[t][1]),
                                           __builtin_fmaxf(acc[t][2], acc[t][3])) > lim;
                }
                const uint64_t any = __builtin_amdgcn_ballot_w64(anyl);
                if (any) {
#pragma unroll
                    for (int v = 0; v < kFV; ++v) hit[v] = acc[t][v] > lim && (!EDGE || jl + v < (uint32_t)a.N);
                    if (f.n + kFV * __builtin_popcountll(any) > kFCandCap) flush(a, f, lane);
                    const uint32_t hi = ((uint32_t)r << a.s_row) | ((uint32_t)(k - 1) << a.s_bin);
                    const int n0 = f.n;
#pragma unroll
                    for (int v = 0; v < kFV; ++v) {
                        const uint64_t mv = __builtin_amdgcn_ballot_w64(hit[v]);
                        if (mv) {
                            const int pre = (int)__builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(mv >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mv, 0));
                            if (hit[v])
                                f.buf[f.n + pre] = ((uint64_t)__float_as_uint(acc[t][v] * a.inv_scale) << 32) |
                                                   (hi | (jl + v));
                            f.n += __builtin_popcountll(mv);
                        }
                    }
                    if (lane == 0) atomicAdd(&f.cnt[k - 1], (uint32_t)(f.n - n0));
                }
            } else {
                float* dst = a.hp + ((int64_t)(k - 1) * a.T + r) * a.N + jl;
                float y[kFV];
#pragma unroll
                for (int v = 0; v < kFV; ++v) y[v] = acc[t][v] * a.inv_scale;
                if constexpr (EDGE) {
#pragma unroll
                    for (int v = 0; v < kFV; ++v)
                        if (jl + v < (uint32_t)a.N) dst[v] = y[v];
                } else {
                    store4(dst, y);
                }
            }
        });
        e = e + 1 < K ? e + 1 : 0;
        changed = (uint32_t)rows::opaque_s((int)row_steps<K, true>(e));
        rows::static_for<1, K>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if (changed & (1u << (m - 1))) at[m] += ldb;
        });
    }
}

// G: planes up to 8 G.
template <typename TIn, bool DETECT, int G>
__device__ __forceinline__ void walk_units(const FracArgs& a, void* smem)
{
    constexpr int W = frac_waves(G);
    const int lane = threadIdx.x & 63;
    const int wave = rows::uni(threadIdx.x >> 6);
    uint64_t* const cand = static_cast<uint64_t*>(smem);
    uint32_t* const cnt = reinterpret_cast<uint32_t*>(cand + (DETECT ? W * kFCandCap : 0));
    if constexpr (DETECT) {
        if ((int)threadIdx.x < kMaxH) cnt[threadIdx.x] = 0;
        __syncthreads();
    }
    Found f{cand + (DETECT ? wave * kFCandCap : 0), cnt, 0};

    // an equal run of the units (strip, rows, chain) for each XCD
    const int xcd = blockIdx.x & 7;
    const int64_t u1 = a.units * (xcd + 1) / 8;
    const int64_t step = (int64_t)((gridDim.x + 7 - xcd) / 8) * W;
    const uint32_t turn = step >= a.groups ? (uint32_t)(step / a.groups) : 1u;
    for (int64_t u = a.units * xcd / 8 + (int64_t)(blockIdx.x >> 3) * W + wave; u < u1; u += step) {
        const uint32_t rest = (uint32_t)(u / a.groups);
        // (turned from one round of the grid to the next, as the chains differ
        // in length)
        const int group = (int)(((uint32_t)(u - (int64_t)rest * a.groups) + rest / turn) % (uint32_t)a.groups);
        const int strip = (int)(rest / (uint32_t)a.pieces);
        const int r0 = (int)(rest - (uint32_t)strip * (uint32_t)a.pieces) * a.rows;
        const int r1 = r0 + a.rows < a.T ? r0 + a.rows : a.T;
        const int j0 = strip * kFBins;
        const bool edge = j0 + kFBins > a.N;
        const int K = a.H - group;
#define HS_CHAIN(k)                                                                       \
    case k:                                                                               \
        if (edge) chain<TIn, k, DETECT, true>(a, f, j0, r0, r1, lane);                    \
        else chain<TIn, k, DETECT, false>(a, f, j0, r0, r1, lane);                        \
        break;
        if constexpr (G == 1) {
            switch (K) {
                HS_CHAIN(1)
                HS_CHAIN(2)
                HS_CHAIN(3)
                HS_CHAIN(4)
                HS_CHAIN(5)
                HS_CHAIN(6)
                HS_CHAIN(7)
                HS_CHAIN(8)
            }
        } else {
            switch (K) {
                HS_CHAIN(5)
                HS_CHAIN(6)
                HS_CHAIN(7)
                HS_CHAIN(8)
                HS_CHAIN(9)
                HS_CHAIN(10)
                HS_CHAIN(11)
                HS_CHAIN(12)
                HS_CHAIN(13)
                HS_CHAIN(14)
                HS_CHAIN(15)
                HS_CHAIN(16)
            }
        }
#undef HS_CHAIN
    }

    if constexpr (DETECT) {
        // the block's last candidates with one atomic
        int* const book = reinterpret_cast<int*>(cnt + kMaxH);
        unsigned long long* const start = reinterpret_cast<unsigned long long*>(book + W);
        if (lane == 0) book[wave] = f.n;
        __syncthreads();
        if (threadIdx.x == 0) {
            int s = 0;
            for (int w = 0; w < W; ++w) s += book[w];
            *start = s ? atomicAdd(&a.counts[a.H], (unsigned long long)s) : 0ull;
        }
        if ((int)threadIdx.x < a.H && cnt[threadIdx.x])
            atomicAdd(&a.counts[threadIdx.x], (unsigned long long)cnt[threadIdx.x]);
        __syncthreads();
        unsigned long long base = *start;
        for (int w = 0; w < wave; ++w) base += (unsigned long long)book[w];
        put(a, f, base, lane);
    }
}

constexpr int frac_lds(bool detect, int G)
{
    return detect ? frac_waves(G) * kFCandCap * 8 + kMaxH * 4 + frac_waves(G) * 4 + 8 : 8;
}

// H <= 8
template <typename TIn, bool DETECT>
__global__ __launch_bounds__(64 * frac_waves(1), frac_occ(1)) void k_frac(FracArgs a)
{
    __shared__ __align__(16) unsigned char smem[frac_lds(DETECT, 1)];
    walk_units<TIn, DETECT, 1>(a, smem);
}

// H > 8
template <typename TIn, bool DETECT>
__global__ __launch_bounds__(64 * frac_waves(2), frac_occ(2)) void k_frac16(FracArgs a)
{
    __shared__ __align__(16) unsigned char smem[frac_lds(DETECT, 2)];
    walk_units<TIn, DETECT, 2>(a, smem);
}

template <typename TIn, bool DETECT>
hipError_t launch_frac_t(FracArgs a, hipStream_t s)
{
    const auto k = a.H <= 8 ? k_frac<TIn, DETECT> : k_frac16<TIn, DETECT>;
    const int W = frac_waves(a.H <= 8 ? 1 : 2);
    int64_t grid = rows::resident_blocks((const void*)k, 64 * W, 0);
    const int64_t strips = ((int64_t)a.N + kFBins - 1) / kFBins;
    // Units (strip, rows, chain): tall enough for sources to be kept from row
    // to row (85 x 2^19 at H = 8: 303 us with one row at a time, 213 with 8,
    // 207 with 16, 215 with 32, whose last units end apart), but kFUnits for
    // every wave while there are rows (21 x 65536: 18.5 us with 6, 17.3 with
    // 3, 15.9 with 1; 33 x 50000 at H = 16: 33, 35 and 38 us).
    a.groups = a.H - a.H / 2;
    int64_t pieces = (kFUnits * W * grid + strips * a.groups - 1) / (strips * a.groups);
    if (pieces > a.T) pieces = a.T;
    a.rows = (int)((a.T + pieces - 1) / pieces);
    if (a.rows > kFRows) a.rows = kFRows;
    a.pieces = (a.T + a.rows - 1) / a.rows;
    a.units = strips * a.pieces * a.groups;
    const int64_t most = 8 * ((a.units + 8 * W - 1) / (8 * W));
    if (grid > most) grid = most;
    if (grid < 8) grid = 8;
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64 * W), 0, s, a);
    return hipGetLastError();
}

template <typename TIn>
hipError_t launch_frac_d(bool detect, const FracArgs& a, hipStream_t s)
{
    return detect ? launch_frac_t<TIn, true>(a, s) : launch_frac_t<TIn, false>(a, s);
}

}  // namespace

hipError_t launch_frac(int dtype, bool detect, const FracArgs& a, hipStream_t s)
{
    if (a.H < 1 || a.H > kMaxH || a.T < 1 || a.N < 1) return hipErrorInvalidValue;
    switch (dtype) {
    case HS_DTYPE_F32: return launch_frac_d<float>(detect, a, s);
    case HS_DTYPE_F16: return launch_frac_d<_Float16>(detect, a, s);
    case HS_DTYPE_BF16: return launch_frac_d<bf16_t>(detect, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace hsk
