// Row walk of one wave: the harmonic planes (Eq. 1-2 of arXiv:1805.12258,
// Sec. III) of a strip of 64 V bins, row after row, thresholded into packed
// candidates, with nothing staged and no plane written to memory.  The
// detection kernels (hs_fused_impl.h, hs_walk_impl.h) differ in the bins per
// lane; the walk is the same.
//
// Registers hold what a row needs.  A lane owns V consecutive bins.  For
// each stretch factor m >= 2 its bins read the source elements floor(j/m)
// of source row floor(i/m): at most two elements for V = 4 and four for
// V = 8, one vector load per lane, selected per bin when the source row
// changes and kept for the m rows that use it.  A row then costs V (H - 1)
// adds, the maximum of the lane's sums per plane and one compare (82 vector
// instructions per row of 256 bins at H = 8).
//
// Loads.  The next source row of every factor is requested when the current
// one is taken into use, i.e. m rows ahead, and a row's own values (m = 1)
// two rows ahead, so a wave always has loads in flight and needs no LDS
// staging, no DMA and no counted wait.
//
// What bounds it (85 x 2^21, H = 8, fp32): the caches' traffic.  The L2s
// fetch 1.51 planes (1.08 GB; 10 % of the requests hit, the sources of one
// strip being read some 20 rows before or after its own rows), which at 169
// us is 6.4 TB/s; vector instructions issue 62 % of the time.  The same plane
// staged tile by tile through LDS took 215 us a call at four waves per SIMD,
// 176 so (fp16 175 and 131; H = 16 355 and 250).  Streaming loads outside the
// source quarter, two rows per step with everything requested two rows
// earlier, and equal shares of rows instead of strips were not faster.
//
// Thresholds come from a small LDS table (one broadcast read per row), which
// also holds the row's bit set of factors whose source row changes there.
//
// Candidates are appended to a private LDS buffer (ballot + mbcnt) and
// counted per plane in LDS; a full buffer is written out with one atomic that
// reserves its places in the list, and the counters are added at the end, one
// atomic per plane and block (batched: per wave and FOP).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "hs_internal.h"

namespace hsk {

struct bf16_t {
    uint16_t bits;
};

namespace rows {

// Entries of a wave's candidate buffer: at least the 64 V hits of one plane
// of a row, which it is given room for at once.
__host__ __device__ static constexpr int cand_cap(int V) { return V == 8 ? 576 : 320; }

typedef const __attribute__((address_space(1))) char* gptr_t;

template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B <= E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// The value of lane 0: states a wave-uniform value as such.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uni64(int64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// x, as a value the compiler knows nothing about (and so forms nothing from
// it ahead of time).
template <typename X>
__device__ __forceinline__ X opaque(X x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// The same for a wave-uniform value.
__device__ __forceinline__ int opaque_s(int x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// A wave-uniform address, kept in scalar registers (the lane's part is then
// the load's 32-bit offset).
__device__ __forceinline__ gptr_t scalar(gptr_t p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// x in a register of its own: a value taken straight from a register that a
// load refills would share it, and the copies that then keep the two apart
// wait for the load.
__device__ __forceinline__ float own(float x)
{
    float y;
    asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
    return y;
}

// Floor division of a (possibly negative) row offset by the constant m:
// shifted into the unsigned range first, so that it is a multiply-high.
template <int m>
__device__ __forceinline__ int floordiv_c(int a)
{
    constexpr uint32_t K = (uint32_t)m * (1u << 21);
    return (int)(((uint32_t)a + K) / (uint32_t)m) - (1 << 21);
}

// f(integral_constant<int, m>) for every m in 2..H whose bit is set in fl,
// four factors tested at a time first: most rows change few factors.
template <int H, typename F>
__device__ __forceinline__ void for_changed(uint32_t fl, F&& f)
{
    static_for<0, (H - 2) / 4>([&](auto gc) {
        constexpr int lo = 2 + 4 * decltype(gc)::value;
        constexpr int hi = lo + 3 < H ? lo + 3 : H;
        constexpr uint32_t gmask = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
        if (fl & gmask) {
            static_for<lo, hi>([&](auto mc) {
                if (fl & (1u << decltype(mc)::value)) f(mc);
            });
        }
    });
}

// A vector of W words in global memory, aligned to at least A bytes.
template <int W, int A> struct Words;
#define HS_WORDS(W, A)                                                  \
    template <> struct Words<W, A> {                                    \
        typedef uint32_t v __attribute__((ext_vector_type(W)));         \
        typedef v m __attribute__((aligned(A)));                        \
    };
HS_WORDS(2, 2) HS_WORDS(2, 4) HS_WORDS(3, 4) HS_WORDS(4, 4) HS_WORDS(2, 8) HS_WORDS(4, 16)
#undef HS_WORDS
typedef uint32_t word_a2 __attribute__((aligned(2)));

// W 32-bit words from p (W = 0: one 16-bit element, in the low half).
template <int W, int A>
__device__ __forceinline__ void load_words(gptr_t p, uint32_t* r)
{
    if constexpr (W == 0) {
        r[0] = *reinterpret_cast<const __attribute__((address_space(1))) uint16_t*>(p);
    } else if constexpr (W == 1) {
        if constexpr (A >= 4) r[0] = *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(p);
        else r[0] = *reinterpret_cast<const __attribute__((address_space(1))) word_a2*>(p);
    } else {
        typedef const __attribute__((address_space(1))) typename Words<W, A>::m* wp_t;
        const typename Words<W, A>::v x = *reinterpret_cast<wp_t>(p);
#pragma unroll
        for (int i = 0; i < W; ++i) r[i] = x[i];
    }
}

// Element e of raw storage words as fp32 (exact).
template <typename TIn>
__device__ __forceinline__ float decode(const uint32_t* r, int e)
{
    if constexpr (std::is_same<TIn, float>::value) {
        return __uint_as_float(r[e]);
    } else if constexpr (std::is_same<TIn, _Float16>::value) {
        const uint16_t b = (uint16_t)(r[e >> 1] >> (16 * (e & 1)));
        _Float16 h;
        __builtin_memcpy(&h, &b, 2);
        return (float)h;
    } else {
        return __uint_as_float((e & 1) ? (r[e >> 1] & 0xffff0000u) : (r[e >> 1] << 16));
    }
}

// Source elements a lane reads for factor m: its V bins start at a multiple
// of V, so when m divides V they cover V/m elements and when V divides m
// one; otherwise bin v reads element (j mod m + v) / m of the lane's range.
__host__ __device__ constexpr int src_elems(int m, int V)
{
    return V % m == 0 ? V / m : (m % V == 0 ? 1 : (m + V - 2) / m + 1);
}
// Values kept per factor: one per group of bins that share an element.
__host__ __device__ constexpr int src_vals(int m, int V) { return m % V == 0 ? 1 : (V % m == 0 ? V / m : V); }
// Whether the elements are selected per bin.
__host__ __device__ constexpr bool src_select(int m, int V) { return V % m != 0 && m % V != 0; }
// Words loaded for them (0: one 16-bit element).  Three 16-bit elements are
// read as four: the lane's row holds at least V - 1 elements past the last.
__host__ __device__ constexpr int src_words(int m, int V, int EB)
{
    return EB == 4 ? src_elems(m, V) : (src_elems(m, V) == 1 ? 0 : (src_elems(m, V) + 1) / 2);
}
// The factor whose source offset stands for m's: floor(j/m) for m = b 2^s is
// floor(floor(j/b) / 2^s), so only the odd b keep a register (b = 1: the bin
// itself).
__host__ __device__ constexpr int odd_part(int m) { return m & 1 ? m : odd_part(m / 2); }
// Place of m's j mod m (four bits) in the packed words, eight to a word.
__host__ __device__ constexpr int sel_slot(int m, int V)
{
    int n = 0;
    for (int k = 2; k < m; ++k) n += src_select(k, V) ? 1 : 0;
    return n;
}

typedef float f4_t __attribute__((ext_vector_type(4), may_alias));
typedef int seg_t __attribute__((ext_vector_type(4), may_alias));

// LDS row table: per row the H thresholds (storage units) and the bit set of
// factors whose source row starts there.
__host__ __device__ static constexpr int tab_stride(int H) { return (H + 1 + 3) & ~3; }

// Rows [row0, row0 + n) of the table by `threads` threads; `t` is the
// calling thread.  Rows past T are zero (the walk reads up to two rows ahead).
template <int H>
__device__ __forceinline__ void build_table(float* tab, int row0, int n, int T, int c, const float* ta, float scale,
                                            int t, int threads)
{
    constexpr int HS = tab_stride(H);
    for (int e = t; e < n * HS; e += threads) {
        const int q = e / HS, k = e - q * HS;
        const int r = row0 + q;
        float v = 0.0f;
        if (r < T) {
            if (k < H) {
                v = ta[(int64_t)k * T + r] * scale;       // exact: the scale is a power of two
            } else if (k == H) {
                uint32_t fl = 0;
#pragma unroll
                for (int m = 2; m <= H; ++m)
                    if ((r - c) % m == 0) fl |= 1u << m;
                v = __uint_as_float(fl);
            }
        }
        tab[e] = v;
    }
}

// Bins a lane sums at a time for strips of 64 V bins: above eight planes the
// values of eight bins would not fit the registers, so a strip of V = 8 is
// walked as two halves.
__host__ __device__ static constexpr int lane_bins(int H, int V) { return H > 8 && V == 8 ? 4 : V; }

// Occupancy asked of the compiler (waves per SIMD): the registers of the
// values in use (about 80 at H = 8, V = 4 and 128 at H = 16, without scratch
// in the row loop).  Measured on 85 x 2^21, hs_detect, H = 8: 171 us at six
// waves, 174 at five.
__host__ __device__ static constexpr int min_waves(int H, int V)
{
    return H <= 4 ? 6 : (H <= 8 ? (V <= 4 ? 6 : 4) : (V <= 4 ? 4 : 3));
}
// Waves per block: a divisor of the waves of a compute unit, and as few
// blocks as that leaves, because every block ends with one atomic per plane
// on the same few counters (about 8 ns a block: 85 x 2^18, H = 8 takes 31 us
// with 768 blocks of eight waves and 40 with 1536 of four; with twelve waves
// the last waves of a block hold its place longer, 185 against 171 us at
// 2^21).
__host__ __device__ static constexpr int block_waves(int H, int V) { return min_waves(H, V) % 2 ? 4 : 8; }

// Block bookkeeping of finish_block (ints).
__host__ __device__ static constexpr int book_ints(int H, int W) { return (W * (H + 1) + 2 + 3) & ~3; }

// A wave's place in a batch: its FOP, and the units of the list that are that
// FOP's.
struct state_t {
    int64_t ld, ubeg, uend;
    uintptr_t fop;
    int32_t N, n, eoff, f;        // bins; strips; first entry; number, -1: none yet
};
static_assert(sizeof(state_t) % 16 == 0, "the table behind it is read 16 bytes at a time");

// The row table covers the plane's rows once per block where it is small,
// else the rows of each wave's piece (at most kOwnRows of them).
constexpr int kTabBytes = 20 * 1024;
constexpr int kOwnRows = 32;
__host__ __device__ static constexpr bool tab_whole(int T, int H) { return (int64_t)(T + 2) * tab_stride(H) * 4 <= kTabBytes; }
__host__ __device__ static constexpr int lds_bytes(int T, int H, int V)
{
    const int W = block_waves(H, V);
    const int tab_rows = tab_whole(T, H) ? T + 2 : W * (kOwnRows + 2);
    return W * (cand_cap(V) * 8 + (int)sizeof(state_t)) + book_ints(H, W) * 4 + tab_rows * tab_stride(H) * 4;
}

// Blocks the device holds at once, at most so many per compute unit.
static inline int resident_blocks(const void* k, int threads, int lds, int most = INT32_MAX)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, threads, lds) != hipSuccess || per_cu < 1) per_cu = 1;
    return cus * std::min(per_cu, most);
}

// Where a wave's candidates go.
struct Sink {
    hs_cand* out;
    int64_t cap;
    unsigned long long* counts;   // [H + 1]
};

template <typename TIn, int H, int V>
struct Walk {
    static constexpr int EB = sizeof(TIn);
    static constexpr int B = 64 * V;
    static constexpr int XW = V * EB / 4;              // words of a lane's row values
    static constexpr bool kSplitX = EB == 4 && V == 8; // two 16-byte loads
    static constexpr int HS = tab_stride(H);
    static constexpr int W = block_waves(H, V);        // waves of the block

    int lane;
    uint64_t* cbuf;               // [cand_cap(V)] LDS
    float inv_scale;
    int s_row, s_bin;
    Sink sink;
    int n;                        // buffered candidates (wave-uniform)
    int* cnt;                     // [H + 1] LDS: the wave's candidates per plane (entry H: finish_block)

    __device__ __forceinline__ Walk(uint64_t* cb, int* ct, float inv, int sr, int sb)
        : lane(threadIdx.x & 63), cbuf(cb), inv_scale(inv), s_row(sr), s_bin(sb), n(0), cnt(ct)
    {
        if (lane <= H) cnt[lane] = 0;
    }

    // Entries [0, m) of the buffer to list positions base + e; those past
    // the capacity are dropped.
    __device__ __forceinline__ void store(int m, unsigned long long base)
    {
        for (int e0 = 0; e0 < m; e0 += 64) {
            const int e = e0 + lane;
            if (e < m && (int64_t)(base + e) < sink.cap) reinterpret_cast<uint64_t*>(sink.out)[base + e] = cbuf[e];
        }
    }

    __device__ __forceinline__ void flush()
    {
        if (n == 0) return;
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&sink.counts[H], (unsigned long long)n);
        store(n, (unsigned long long)uni64((int64_t)base));
        n = 0;
    }

    // Everything of this FOP out, one wave on its own.
    __device__ __forceinline__ void finish_wave()
    {
        flush();
        if (lane < H && cnt[lane]) atomicAdd(&sink.counts[lane], (unsigned long long)cnt[lane]);
        if (lane < H) cnt[lane] = 0;
    }

    // The same for the block's waves together (all of them call it): one
    // atomic per counter for the block.  book: the waves' counters, then two
    // ints.
    __device__ __forceinline__ void finish_block(int* book)
    {
        const int wave = uni(threadIdx.x >> 6);
        if (lane == 0) cnt[H] = n;
        __syncthreads();
        int* const res = book + W * (H + 1);
        if (threadIdx.x <= H) {
            int s = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) s += book[w * (H + 1) + threadIdx.x];
            unsigned long long b = 0;
            if (s) b = atomicAdd(&sink.counts[threadIdx.x], (unsigned long long)s);
            if (threadIdx.x == H) {
                res[0] = (int)(uint32_t)b;
                res[1] = (int)(uint32_t)(b >> 32);
            }
        }
        __syncthreads();
        unsigned long long base = ((unsigned long long)(uint32_t)res[1] << 32) | (uint32_t)res[0];
        for (int w = 0; w < wave; ++w) base += (unsigned long long)book[w * (H + 1) + H];
        store(n, base);
    }

    // Hits of plane k among the lane's sums (the rare path, whole wave; the
    // buffer has room for them).
    template <int k>
    __device__ __forceinline__ void emit(const float (&acc)[V], float tk, int row, int jb)
    {
        const int r = opaque_s(row);
        const uint32_t hi = (uint32_t)(((uint64_t)r << s_row) | ((uint64_t)(k - 1) << s_bin));
        const int j = opaque(jb);        // the words are formed here, not ahead for every plane
        const int n0 = n;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const bool hit = acc[v] > tk;
            const uint64_t mk = __builtin_amdgcn_ballot_w64(hit);
            if (mk) {
                const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0));
                const float pw = EB == 4 ? acc[v] : acc[v] * inv_scale;   // unscaled power
                if (hit) cbuf[n + pre] = ((uint64_t)__float_as_uint(pw) << 32) | (hi | (uint32_t)(j + v));
                n += __builtin_popcountll(mk);
            }
        }
        if (lane == 0) cnt[k - 1] += n - n0;
    }

    // One unit: rows [r0, r1) of the strip at bin j0 (j0 < N) of a plane of
    // N bins and row pitch ld elements (whole multiples of 16 bytes).  tab:
    // the LDS row table, whose first row is plane row trow0.
    __device__ __forceinline__ void unit(gptr_t fop_, int64_t ld_, int N_, int c, int j0_, int r0_, int r1_,
                                         const float* tab, int trow0)
    {
        // wave-uniform values, stated as such for the compiler
        const gptr_t fop = (gptr_t)(uintptr_t)uni64((int64_t)(uintptr_t)fop_);
        const int64_t ld = uni64(ld_);
        const int N = uni(N_), j0 = uni(j0_), r0 = uni(r0_), r1 = uni(r1_);
        const int64_t ldb = ld * EB;
        const int jb = j0 + V * lane;
        const int over = uni(j0 + B - N);     // bins of the strip past the plane's last
        // lanes past the last bin re-read the last group of V bins
        const int jc = min(jb, (N - 1) / V * V);
        const uint32_t vx = (uint32_t)(jc - j0) * EB;
        uint32_t vx2 = 0;
        if constexpr (kSplitX) vx2 = (int64_t)jc + 8 <= ld ? vx + 16 : vx;

        const gptr_t xbase = fop + (int64_t)j0 * EB;
        uint32_t vq[H + 1];             // floor(j / b) of odd b at the lane's first bin
        uint32_t rm[2] = {0, 0};        // j mod m, packed
        uint32_t raw[H + 1][4];         // the next source row's elements, in flight
        float sv[H + 1][V];             // values in use

        auto load_x = [&](int r, uint32_t (&x)[XW]) __attribute__((always_inline)) {
            const gptr_t p = scalar(xbase + r * ldb);
            load_words<kSplitX ? 4 : XW, kSplitX ? 16 : XW * 4>(p + opaque(vx), x);
            if constexpr (kSplitX) load_words<4, 16>(p + opaque(vx2), x + 4);
        };
        // the source elements of the row that plane row r reads (r < r1)
        const int last = r1 - 1;
        auto load_src = [&](auto mc, int r, uint32_t (&w)[4]) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            const int sr = floordiv_c<m>(min(r, last) - c) + c;
            // the element floor(j / m), formed anew (below 2^32 bytes: j / m <= 2^30)
            constexpr int b = odd_part(m);
            const uint32_t q = opaque(vq[b]) / (uint32_t)(m / b);
            load_words<src_words(m, V, EB), EB>(scalar(fop + sr * ldb) + q * EB, w);
        };
        auto take_src = [&](auto mc, const uint32_t (&w)[4]) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            constexpr int NE = src_elems(m, V);
            float e[NE];
#pragma unroll
            for (int q = 0; q < NE; ++q) e[q] = decode<TIn>(w, q);
            if constexpr (!src_select(m, V)) {
#pragma unroll
                for (int q = 0; q < NE; ++q) sv[m][q] = own(e[q]);
            } else {
                // compared anew each time: kept across rows, the masks of all
                // factors would not fit the scalar registers
                constexpr int slot = sel_slot(m, V);
                const int j = (int)((opaque(rm[slot / 8]) >> (4 * (slot % 8))) & 15u);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const int lo = v / m, hi = (m - 1 + v) / m;     // hi <= lo + 1
                    sv[m][v] = lo == hi ? own(e[lo]) : (j >= hi * m - v ? e[hi] : e[lo]);
                }
            }
        };

        vq[1] = (uint32_t)jc;
        static_for<2, H>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const uint32_t q = (uint32_t)jc / (uint32_t)m;
            if constexpr (m & 1) vq[m] = q;
            if constexpr (src_select(m, V)) rm[sel_slot(m, V) / 8] |= ((uint32_t)jc - q * m) << (4 * (sel_slot(m, V) % 8));
        });
        static_for<2, H>([&](auto mc) { load_src(mc, r0, raw[decltype(mc)::value]); });
        uint32_t xa[XW], xb[XW];
        load_x(r0, xa);
        load_x(min(r0 + 1, last), xb);
        const float* tr = tab + (r0 - trow0) * HS;
        static_for<2, H>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            take_src(mc, raw[m]);
            load_src(mc, r0 + m, raw[m]);
        });
        uint32_t fl = 0;                // factors that change at this row

        // one row from x, whose registers row r + 2 takes.  The order of the
        // waits: a row's values are taken before its new source rows are
        // requested, and those before row r + 2, so that what is waited for
        // (loads complete in order) is never younger than one row.
        auto row = [&](int r, uint32_t (&x)[XW]) __attribute__((always_inline)) {
            float acc[V];
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = own(decode<TIn>(x, v));
            if constexpr (H >= 2) {
                for_changed<H>(fl, [&](auto mc) {
                    constexpr int m = decltype(mc)::value;
                    take_src(mc, raw[m]);
                    load_src(mc, r + m, raw[m]);
                });
            }
            load_x(min(r + 2, last), x);
            float t[HS];
#pragma unroll
            for (int k = 0; k < HS; k += 4) {
                const f4_t q = *reinterpret_cast<const f4_t*>(tr + k);
                t[k] = q.x; t[k + 1] = q.y; t[k + 2] = q.z; t[k + 3] = q.w;
            }
            tr += HS;
            const float fn = H >= 2 ? tr[H] : 0.0f;      // next row's changes
            // planes from kbeg on are emitted; when one finds no room in the
            // buffer (kfull), the buffer is written out and the row formed
            // again, from its values read anew, for the planes from that one on
            int kbeg = r < r1 ? 1 : H + 1;
            n = uni(n);
            for (;;) {
                int kfull = 0;
                auto detect = [&](auto kc) __attribute__((always_inline)) {
                    constexpr int k = decltype(kc)::value;
                    float mx = acc[0];
#pragma unroll
                    for (int v = 1; v < V; ++v) mx = fmaxf(mx, acc[v]);
                    const uint64_t any = __builtin_amdgcn_ballot_w64(mx > t[k - 1]);
                    if (__builtin_expect(any != 0, 0)) {
                        if (k >= kbeg && kfull == 0) {
                            if (uni(n) + V * __builtin_popcountll(any) > cand_cap(V)) kfull = k;
                            else emit<k>(acc, t[k - 1], r, jb);
                        }
                    }
                };
                if (opaque_s(over) > 0) {
                    // bins past the end start at -inf: no sum of them passes a threshold
                    const int j = opaque(jb);
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] = j < N - v ? acc[v] : -__builtin_inff();
                }
                detect(std::integral_constant<int, 1>{});
                static_for<2, H>([&](auto mc) {
                    constexpr int m = decltype(mc)::value;
                    constexpr int NV = src_vals(m, V);
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        acc[v] = acc[v] + (NV == 1 ? sv[m][0] : (NV < V ? sv[m][v / m] : sv[m][v]));
                    detect(mc);
                });
                if (__builtin_expect(kfull == 0, 1)) break;
                flush();
                kbeg = kfull;
                uint32_t y[XW];
                load_x(opaque_s(r), y);
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = own(decode<TIn>(y, v));   // waits here, in the rare path
            }
            if constexpr (H >= 2) fl = (uint32_t)uni(__float_as_int(fn));
        };
        // rows in pairs with one way out (an exit between the two would make
        // the first row's wait cover the loads just issued); a row past the
        // last forms sums that nothing is emitted from
        for (int r = r0; r < r1; r += 2) {
            row(r, xa);
            row(r + 1, xb);
        }
    }
};

// Detection over the units of a plan.  A strip's rows are cut at template
// index 0 (under the floor of Eq. 1 the two halves read disjoint source rows:
// floor(i/m) keeps the sign of i), each half into a.pieces runs; the units of
// a segment of strips are all pieces of the lower halves, then those of the
// upper ones, so that the source rows in use at one time are those of one
// half.  The waves on an XCD take its units in turn (all waves those of the one
// list of a plane of few strips).
template <typename TIn, int H, int V, bool BATCH>
__device__ __forceinline__ void walk_plan(const WalkArgs& a, unsigned char* smem)
{
    constexpr int EB = sizeof(TIn);
    constexpr int VI = lane_bins(H, V);
    constexpr int W = block_waves(H, VI);
    constexpr int HS = tab_stride(H);
    uint64_t* const cands = reinterpret_cast<uint64_t*>(smem);
    int* const book = reinterpret_cast<int*>(cands + W * cand_cap(VI));
    state_t* const states = reinterpret_cast<state_t*>(book + book_ints(H, W));
    float* tab = reinterpret_cast<float*>(states + W);
    const int wave = uni(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const bool whole = tab_whole(a.T, H);
    const bool shared = a.lists == 1;
    const int xcd = shared ? 0 : blockIdx.x & 7;
    const int nw = (int)(shared ? gridDim.x : (gridDim.x - xcd + 7) >> 3) * W;       // waves on this list
    int64_t at = (int64_t)((int)(shared ? blockIdx.x : blockIdx.x >> 3) * W + wave) * a.run;
    const int halves = a.c > 0 ? 2 : 1;
    auto split = [&](int64_t u, int n, int& q, int& p) __attribute__((always_inline)) {
        const bool up = u >= (int64_t)n * a.pieces;
        if (up) u -= (int64_t)n * a.pieces;
        q = uni((int)(u / a.pieces));
        p = uni((int)(u - (int64_t)q * a.pieces));
        return up;
    };
    // first strip of a single FOP (its XCD lists are in the arguments),
    // requested before the table is waited for
    int strip = -1;
    if constexpr (!BATCH) {
        if (at < (int64_t)a.xcount[xcd] * halves * a.pieces) {
            int q, p;
            split(at, a.xcount[xcd], q, p);
            strip = (int)a.ent[a.xfirst[xcd] + q];
        }
    }
    if (whole) build_table<H>(tab, 0, a.T + 2, a.T, a.c, a.ta, a.scale, threadIdx.x, 64 * W);
    else tab += wave * (kOwnRows + 2) * HS;
    __syncthreads();
    strip = uni(strip);

    Walk<TIn, H, VI> w(cands + wave * cand_cap(VI), book + wave * (H + 1), a.inv_scale, a.s_row, a.s_bin);
    // piece p of the lower or upper half of the strip at entry value e
    auto one = [&](gptr_t fop, int64_t ld, int N, bool up, int p, uint32_t e) __attribute__((always_inline)) {
        // runs of even length (the walk takes two rows at a time); the last may be empty
        const int h0 = up ? a.c : 0, h1 = up || halves == 1 ? a.T : a.c;
        const int len = ((h1 - h0 + a.pieces - 1) / a.pieces + 1) & ~1;
        const int r0 = min(h0 + p * len, h1), r1 = min(r0 + len, h1);
        if (r0 >= r1) return;
        if (!whole) build_table<H>(tab, r0, r1 - r0 + 2, a.T, a.c, a.ta, a.scale, lane, 64);
        const int64_t j0 = (int64_t)(uint32_t)uni((int)e) * (64 * V);
#pragma unroll 1
        for (int64_t j = j0; j < N && j < j0 + 64 * V; j += 64 * VI)
            w.unit(fop, ld, N, a.c, (int)j, r0, r1, tab, whole ? 0 : r0);
    };

    if constexpr (!BATCH) {
        w.sink = Sink{a.out, a.cap, a.counts};
        const int n = a.xcount[xcd];
        const int64_t units = (int64_t)n * halves * a.pieces;
        for (; at < units; at = uni64(at + nw)) {
            w.n = uni(w.n);
            int q, p;
            const bool up = split(at, n, q, p);
            if (strip < 0) strip = uni((int)a.ent[a.xfirst[xcd] + q]);
            one((gptr_t)a.fop, a.ld, a.N, up, p, (uint32_t)strip);
            strip = -1;
        }
        w.finish_block(book);
        return;
    }

    // what the wave needs to know of its FOP lies in LDS from unit to unit: the
    // walk has no scalar registers to spare
    states[wave] = state_t{0, 0, 0, 0, 0, 0, 0, -1};
    for (;;) {
        // wave-uniform loop state, stated as such for the compiler
        at = uni64(at);
        w.n = uni(w.n);
        asm volatile("" ::: "memory");
        state_t& st = states[opaque_s(wave)];
        const state_t now = st;         // (all of it requested before any is waited for)
        if (at >= uni64(now.uend)) {
            // the segment of the list that holds the unit: FOP, first entry,
            // first and end index.  Many short FOPs lie between two units of a
            // wave, so 64 segments are looked at in one step (5000 FOPs of 9 x
            // 100 bins 387 us one after another, 31 so)
            int lo = a.xseg[xcd], hi = a.xseg[xcd + 1], step = 1, before = 0;
            seg_t g;
            const int l = opaque(lane);
            do {
                const int left = uni(hi - lo);
                if (left <= 0) break;
                step = (left + 63) >> 6;
                const int i = lo + (l + 1) * step - 1;
                g = reinterpret_cast<const seg_t*>(a.seg)[min(i, hi - 1)];
                const bool past = i < hi && (int64_t)g.w * halves * a.pieces <= at;
                before = uni(__builtin_popcountll(__builtin_amdgcn_ballot_w64(past)));
                lo = uni(lo + before * step);
                hi = min(hi, lo + step);
            } while (step > 1);
            if (lo >= hi) break;
            const int f = __builtin_amdgcn_readlane(g.x, before);
            const int i0 = __builtin_amdgcn_readlane(g.z, before), n = __builtin_amdgcn_readlane(g.w, before) - i0;
            const int64_t ubeg = (int64_t)i0 * halves * a.pieces;
            const int cur = uni(now.f);
            st.eoff = __builtin_amdgcn_readlane(g.y, before);
            st.n = n;
            st.ubeg = ubeg;
            st.uend = ubeg + (int64_t)n * halves * a.pieces;
            if (f == cur) continue;
            if (cur >= 0 && w.sink.counts) w.finish_wave();
            const uintptr_t fp = (uintptr_t)uni64((int64_t)(uintptr_t)a.fops[f]);
            const int N = uni((int)a.n_chans[f]);
            const int64_t ld = uni64(a.lds[f]);
            st.f = f;
            st.N = N;
            st.ld = ld;
            st.fop = fp;
            // a FOP whose address or pitch breaks the alignment rules is
            // skipped (no counts to add to), its total set to -1
            const bool ok = (fp & 15) == 0 && ld % (16 / EB) == 0 && ld >= N &&
                            ((uint64_t)ld * (uint64_t)a.lim_rows + (uint64_t)a.lim_bins) * EB <= 0xffffffffull;
            unsigned long long* const cn = a.counts + (int64_t)f * (H + 1);
            w.sink = Sink{a.out + uni64(a.out_offsets[f]), uni64(a.caps[f]), ok ? cn : nullptr};
            if (!ok && l == 0) cn[H] = ~0ull;
            continue;
        }
        if (w.sink.counts) {
            int q, p;
            const bool up = split(at - uni64(now.ubeg), uni(now.n), q, p);
            const uint32_t e = (uint32_t)uni((int)a.ent[uni(now.eoff) + q]);
            one((gptr_t)(uintptr_t)uni64((int64_t)now.fop), uni64(now.ld), uni(now.N), up, p, e);
        }
        at += 1;
        if (((int)at & (a.run - 1)) == 0) at += (int64_t)(nw - 1) * a.run;
    }
    // waves may end on different FOPs
    if (uni(states[wave].f) >= 0 && w.sink.counts) w.finish_wave();
}

// Pieces a half strip's rows are cut into, for `strips` strips on `waves`
// resident waves: enough units for two rounds of the waves while a piece
// keeps a third of a half plane of 42 rows (a piece's start costs about two
// exposed latencies), at least one round down to three rows.
static inline int row_pieces(int64_t strips, int T, int64_t waves, bool whole)
{
    const int64_t units = strips * (T > 1 ? 2 : 1);
    const int rows = T > 1 ? (T + 1) / 2 : 1;
    int p = whole ? 1 : (rows + kOwnRows - 1) / kOwnRows;
    while (units * p < 2 * waves && rows / (p + 1) >= 14) ++p;
    while (units * p < waves && rows / (p + 1) >= 3) ++p;
    return p;
}

// Units that a wave of a batch takes one after another.  A wave writes out what
// it found whenever it comes to another FOP, and where FOPs are short (fewer
// units than a list has waves) that is at every unit; runs of units save it
// where units are short too, as long as the last round is not much emptier.
// 100 FOPs of 21 x 50000 at four planes (units of 11 rows, 4900 on a list of 768
// waves): 160 us one by one, 127 by two, 116 by four; 1000 of 85 x 3000 (units of
// 43 rows) 276, 290 and 292.
static inline int unit_run(int64_t units, int64_t waves, int64_t per_fop, int rows)
{
    if (rows > 16 || per_fop > waves) return 1;
    auto rounds = [&](int run) { return (units + waves * run - 1) / (waves * run) * run; };
    return rounds(4) * 4 <= rounds(1) * 5 ? 4 : (rounds(2) * 4 <= rounds(1) * 5 ? 2 : 1);
}

// Launch of a detection kernel k over the plan's units.
template <typename... A>
static hipError_t launch_plan(void (*k)(WalkArgs, A...), int H, int V, WalkArgs a, int grid, hipStream_t s)
{
    const int VI = lane_bins(H, V);
    const int W = block_waves(H, VI);
    const int lds = lds_bytes(a.T, H, VI);
    (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    // the waves the kernel is compiled for, also where few planes leave registers
    // for more: 1024 blocks for 768 cost 85 x 2^18 fp32 at two planes 40 us for
    // 34 (their atomics at the end)
    if (grid <= 0) grid = resident_blocks((const void*)k, 64 * W, lds, 4 * min_waves(H, VI) / W);
    if (grid < a.lists) grid = a.lists;   // every list needs a block
    a.pieces = row_pieces(a.lists * a.units_per_list, a.T, (int64_t)grid * W, tab_whole(a.T, H));
    const int halves = a.T > 1 ? 2 : 1;
    const int64_t units = a.units_per_list * halves * a.pieces;
    a.run = a.n_fops == 0 ? 1 : unit_run(units, (int64_t)grid / a.lists * W, units * a.lists / a.n_fops,
                                         (a.T / halves + a.pieces - 1) / a.pieces);
    const int64_t most = a.lists * ((units + W - 1) / W);
    if (grid > most) grid = (int)most;
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * W), lds, s, a, A{}...);
    return hipGetLastError();
}

}  // namespace rows
}  // namespace hsk
