// Transpose of the plane map (the vector-Jacobian product of Eq. 1-2) and
// the log-sum-exp statistic built on it.
//
// Backward.  With G_m = sum_{k >= m} g_k (suffix sums over the planes),
//     dFOP(a, b) = sum_m  sum_{(r, j) : src(r, m) = a, floor(j/m) = b}  G_m(r, j),
// where src(r, m) = floor((r - c)/m) + c is the source row of Eq. 1.  The
// preimage of (a, b) under m is an m x m box of plane points (clipped to the
// plane).  Two deterministic passes, no floating-point atomics:
//   1. a wave walks a piece of a few rows of a strip of 256 bins, four bins a
//      lane: it takes g_H .. g_1 of a row (read, or formed from the FOP for
//      the statistic), forms the suffix sums in registers, writes G_1 to dFOP
//      and adds G_m, m >= 2, to a register sum over the rows of one target
//      row; when the target row ends (every m rows), the sum over the m bins
//      of each target goes to a per-(m, piece) partial row in the workspace;
//   2. per dFOP point: add, for m = 2..H in order, the partials that cover it
//      (two where its box lies across strips or pieces, at most four above
//      the smallest pieces).
// The same input gives bitwise the same output.  No barrier and little LDS:
// summing down the rows in registers leaves one horizontal sum every m rows
// (m = 2, 4, 8, 16 by lanes alone).
//
// What bounds it.  The plain transpose: memory, 85 x 2^18 at H = 8 reads 713 MB
// and writes 149 in 173 us of a training step (5.0 TB/s).  The statistic's:
// the vector units, 32 exponentials (a quarter of the rate) and 240 other
// instructions per row of 256 bins: 85 x 2^20 230 to 250 us.  The second pass:
// 19 and 79 us.  Both passes together, repeated, 168 and 312 us; tiles of rows
// staged in LDS factor by factor, with a barrier each, and one point per
// thread in the second pass took 325 and 640 us (at H = 16, 85 x 2^18, 770 and
// 908, now 418 and 287).
//
// Log-sum-exp.  lse_k = log sum_{i,j} exp(HP_k(i,j) / tau) per plane, with a
// running maximum (each term exp(x - M) <= 1) and a fixed two-level
// reduction; lse is returned in fp64 so that the weights
// exp(HP_k / tau - lse_k) of the backward keep fp32 accuracy even where
// |lse| is large.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hs_rows.h"

namespace hsk {

namespace {

using rows::gptr_t;
using rows::static_for;

constexpr int kGWaves = 4;                         // waves of a block (independent of each other)
constexpr int kGThreads = kGWaves * kLanes;

struct BwdArgs {
    const void* src;                 // the FOP, or g [H][T][N]
    int64_t ld;                      // of the FOP
    int32_t T, c, N;
    int32_t shift, row_blocks, n_bt; // pieces of 2^shift rows, strips
    float* dfop;
    float* part;
    int64_t off[kMaxH + 1];          // start of the partial rows of m
    // the statistic's weights
    double inv_scale, tau;
    float c2;
    const double* lse;
    const double* gscale;
};

constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

// Elements that four bins from a multiple of four read for m.
constexpr int src_span(int m) { return (m - gcd_c(kV, m) + kV - 1) / m + 1; }

// floor(i / m) for i >= -c (exact for any c >= 0).
template <int m>
__device__ __forceinline__ int floor_div(int i, int c)
{
    const int over = (c + m - 1) / m;
    return (int)((uint32_t)(i + over * m) / (uint32_t)m) - over;
}

// Rows of partial sums that a piece of R rows has for m: the most distinct
// floor(i/m) over R consecutive template indices.
__host__ __device__ constexpr int piece_rows(int R, int m) { return (R + m - 2) / m + 1; }

// A partial row of m: the targets floor(j/m), each with the part of its box in
// the strip where it begins, then for every strip the part of a target that
// began in the strip before (m bins rarely divide 256), so that the targets
// are contiguous for the second pass; four elements more for its loads.
// (in 32 bits without a sign, which hold N + 15; as (N - 1) / m + 1 the second pass
// at 16 planes spills more, and the statistic's 65536 x 256 takes 265 us for 250)
__host__ __device__ inline int targets(int m, int N) { return (int)(((uint32_t)N + (uint32_t)(m - 1)) / (uint32_t)m); }
__host__ __device__ inline int partial_pitch(int m, int N, int n_bt) { return (targets(m, N) + n_bt + 7) & ~3; }

typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// The planes' gradients of a row as they are stored.  NT: by loads that leave
// the caches alone, for planes that are larger than those.  In the last strip
// of a ragged plane the lanes past the end, and the one across it, load the
// row's last four elements; that one takes its own from them (one load a plane
// as elsewhere: with a guarded load per bin the pass took 65536 x 100 at H = 16
// 608 us, 150 so; at H = 8 114 and 43).
template <int H, bool NT>
struct PlaneSource {
    typedef const __attribute__((address_space(1))) float4_a4* q_t;
    const BwdArgs& a;
    int j0;
    bool edge;
    int first;             // bin of the strip that offsets count from (below 0 for a strip of less than four)
    uint32_t off;
    int past;              // elements of the lane's load before its own (4 or more: none of them)

    __device__ __forceinline__ PlaneSource(const BwdArgs& a_, int lane, int j0_, int) : a(a_), j0(j0_)
    {
        edge = j0 + kTileBins > a.N;
        const int last = edge ? a.N - j0 - kV : kTileBins - kV;
        first = min(last, 0);
        const int from = min(kV * lane, last);
        off = (uint32_t)(from - first) * 4u;
        past = kV * lane - from;
    }
    __device__ __forceinline__ float sign() const { return 1.0f; }
    __device__ __forceinline__ void request(int, uint32_t) {}
    __device__ __forceinline__ void weights(int r, float (&G)[H][kV])
    {
        const int64_t plane = (int64_t)a.T * a.N * 4;
        if (a.N < kV) {        // (rows of less than four elements: one strip)
            const int lane = threadIdx.x & 63;
            gptr_t p = (gptr_t)(uintptr_t)a.src + (int64_t)r * a.N * 4;
            static_for<1, H>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
#pragma unroll
                for (int v = 0; v < kV; ++v) {
                    uint32_t x[1];
                    rows::load_words<1, 4>(rows::scalar(p) + (uint32_t)(4 * min(v, a.N - 1)), x);
                    G[k - 1][v] = lane == 0 && v < a.N ? __uint_as_float(x[0]) : 0.0f;
                }
                p += plane;
            });
            return;
        }
        gptr_t p = (gptr_t)(uintptr_t)a.src + ((int64_t)r * a.N + j0 + first) * 4;
        static_for<1, H>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const q_t at = reinterpret_cast<q_t>(rows::scalar(p) + off);
            const float4_a4 t = NT ? __builtin_nontemporal_load(at) : *at;
#pragma unroll
            for (int v = 0; v < kV; ++v) G[k - 1][v] = t[v];
            p += plane;
        });
        if (edge) {
#pragma unroll
            for (int k = 0; k < H; ++k) {
#pragma unroll
                for (int v = 0; v < kV; ++v) {
                    float y = past == 0 ? G[k][v] : 0.0f;
#pragma unroll
                    for (int d = 1; v + d < kV; ++d) y = past == d ? G[k][v + d] : y;
                    G[k][v] = y;
                }
            }
        }
    }
};

// The weights g_k = gscale exp(HP_k / tau - lse_k) of a row, from the FOP:
// HP_1..HP_H in the order of Eq. 2 (the forward's sums, so the weights are
// those of the planes the statistic was taken over), no weight plane stored.
// In base 2 and fp32, with no fp64 operation per point: with L_k = tau lse_k /
// input_scale (fp64, in storage units) split as L_hi + L_lo (two fp32 values,
// L_lo below half an ulp of L_hi),
//     log2 |g_k| = (HP - L_hi) c - L_lo c + log2|gscale|,  c = log2(e) / (tau scale),
// formed as fma(HP - L_hi, c, K_k) with K_k = -L_lo c + log2|gscale| per
// plane.  HP - L_hi is exact where HP is within a factor two of L_hi (the
// weights that matter: lse_k is at least max HP_k / tau), and the remaining
// roundings leave a few fp32 ulps of relative error in the exponent.  The sign
// of gscale is applied to the sums, zero gives zero weights.
//
// A source value m >= 2 is loaded when its row changes (every m rows) and
// kept: at most two elements per lane, one vector load.
template <typename TIn, int H>
struct LseSource {
    static constexpr int EB = sizeof(TIn);
    static constexpr int XW = kV * EB / 4;
    const BwdArgs& a;
    const int64_t ldb;
    bool edge, neg;
    int jl;
    uint32_t vx, q[H + 1], rem[H + 1];
    gptr_t xrow, at[H + 1];
    uint32_t x[XW], raw[H + 1][2];
    float hi[H], kk[H];

    __device__ __forceinline__ LseSource(const BwdArgs& a_, int lane, int j0, int r0) : a(a_), ldb(a_.ld * EB)
    {
        edge = j0 + kTileBins > a.N;
        jl = j0 + kV * lane;
        // lanes past the end read a valid element
        const int last = (a.N - 1) & ~(kV - 1);
        const uint32_t jc = (uint32_t)(jl < last ? jl : last);
        vx = jc * EB;
        xrow = (gptr_t)(uintptr_t)a.src + r0 * ldb;
        static_for<2, H>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const uint32_t e = jc / (uint32_t)m;
            q[m] = e * EB;
            rem[m] = jc - e * (uint32_t)m;
            at[m] = (gptr_t)(uintptr_t)a.src + (floor_div<m>(r0 - a.c, a.c) + a.c) * ldb;
        });
        const double gsc = a.gscale ? *a.gscale : 1.0;
        neg = gsc < 0.0;
        // lane k - 1 forms the constants of plane k
        const int k = lane < H ? lane : H - 1;
        const double L = a.tau * a.lse[k] / a.inv_scale;
        const float h = (float)L;
        const float lo = (float)(L - (double)h);
        const float c0 = (float)(-(double)lo * (double)a.c2 + log2(fabs(gsc)));
#pragma unroll
        for (int i = 0; i < H; ++i) {
            hi[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h), i));
            kk[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c0), i));
        }
    }
    __device__ __forceinline__ float sign() const { return neg ? -1.0f : 1.0f; }
    // the values of the next row; m whose source row begins there are in `fl`
    __device__ __forceinline__ void request(int first, uint32_t fl)
    {
        if (!first) xrow += ldb;
        rows::load_words<XW, XW * 4>(rows::scalar(xrow) + rows::opaque(vx), x);
        static_for<2, H>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int W = src_span(m);
            if (fl & (1u << m)) {
                if (!first) at[m] += ldb;
                rows::load_words<EB == 4 ? W : W - 1, EB>(rows::scalar(at[m]) + rows::opaque(q[m]), raw[m]);
            }
        });
    }
    __device__ __forceinline__ void weights(int, float (&G)[H][kV])
    {
        float acc[kV];
        static_for<1, H>([&](auto kc) {
            constexpr int k = decltype(kc)::value, step = gcd_c(kV, k);   // the remainders' step
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                float y;
                if constexpr (k == 1) {
                    y = rows::decode<TIn>(x, v);
                    acc[v] = y;
                } else {
                    const int lo = v / k, left = v % k;
                    y = rows::decode<TIn>(raw[k], lo);
                    if (left >= step) y = rem[k] >= (uint32_t)(k - left) ? rows::decode<TIn>(raw[k], lo + 1) : y;
                    acc[v] = acc[v] + y;
                }
                G[k - 1][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v] - hi[k - 1], a.c2, kk[k - 1]));
            }
        });
        if (edge) {
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                const bool ok = jl + v < a.N;
#pragma unroll
                for (int k = 0; k < H; ++k) G[k][v] = ok ? G[k][v] : 0.0f;
            }
        }
    }
};

// A wave's row in LDS while its bins are summed over the targets: zero bins on
// both sides (the first target starts up to m - 1 bins before the strip, the
// last column can end up to 23 bins after it for m <= 16), so that the sums
// test no bounds.
constexpr int kGPad = kMaxH;                       // zero bins before the strip
constexpr int kGPadR = 2 * kMaxH;                  // and after it
constexpr int kGPitch = kGPad + kTileBins + kGPadR;

typedef float float2_a4 __attribute__((ext_vector_type(2), aligned(4)));

// x of the lane whose number differs in the bits of `quad` (1 or 2).
template <int quad>
__device__ __forceinline__ float other(float x)
{
    constexpr int sel = quad == 1 ? 0xB1 : 0x4E;   // lanes 1 0 3 2, or 2 3 0 1
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), sel, 0xf, 0xf, true));
}

// The sums of S over the bins of each target of the strip, to the strip's
// place in a partial row.  `end`: bins of the strip before the plane's end;
// `side` is the offset from out[0] of the place for a first target that begins
// in the strip before.
template <int m>
__device__ __forceinline__ void emit_targets(const float (&S)[kV], float* row, int j0, int end, int side, int lane,
                                             float* out)
{
    if constexpr (m == 2) {
        if (kV * lane < end) *reinterpret_cast<float2_a4*>(out + 2 * lane) = float2_a4{S[0] + S[1], S[2] + S[3]};
    } else if constexpr (m == 4 || m == 8 || m == 16) {
        float t = (S[0] + S[1]) + (S[2] + S[3]);
        if constexpr (m >= 8) t += other<1>(t);
        if constexpr (m >= 16) t += other<2>(t);
        if ((lane & (m / 4 - 1)) == 0 && kV * lane < end) out[lane / (m / 4)] = t;
    } else {
        *reinterpret_cast<float4*>(row + kV * lane) = make_float4(S[0], S[1], S[2], S[3]);
        // the wave reads back bins its other lanes wrote: keep the order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int jf = -(j0 % m);                  // first target's first bin
        const float* const s0 = row + jf;
#pragma unroll
        for (int t0 = 0; t0 < stage_pitch(m); t0 += 64) {
            const int tc = t0 + lane;
            if (jf + m * tc < end) {
                const float* src = s0 + m * tc;
                float acc = src[0];
#pragma unroll
                for (int d = 1; d < m; ++d) acc += src[d];
                out[t0 == 0 && tc == 0 && jf < 0 ? side : tc] = acc;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

template <int H, typename Source>
__device__ __forceinline__ void bwd_walk(const BwdArgs& a, float* lds)
{
    const int lane = threadIdx.x & 63;
    const int wave = rows::uni(threadIdx.x >> 6);
    // an equal run of the units (piece, strip) for each XCD: neighbouring waves
    // read neighbouring strips of the same rows
    const int64_t units = (int64_t)a.n_bt * a.row_blocks;
    const int xcd = blockIdx.x & 7;
    const int64_t u = units * xcd / 8 + (int64_t)(blockIdx.x >> 3) * kGWaves + wave;
    if (u >= units * (xcd + 1) / 8) return;
    const int rb = (int)((uint32_t)u / (uint32_t)a.n_bt);
    const int bt = (int)((uint32_t)u - (uint32_t)rb * (uint32_t)a.n_bt);
    const int r0 = rb << a.shift;
    const int r1 = min(r0 + (1 << a.shift), a.T);
    const int j0 = bt * kTileBins;
    const int end = min(a.N - j0, kTileBins);
    float* const row = lds + wave * kGPitch + kGPad;
    if (lane < kGPad) row[lane - kGPad] = 0.0f;
    if (lane < kGPadR) row[kTileBins + lane] = 0.0f;

    // lane l: the m whose target row begins at row r0 + l (bit m)
    uint32_t begins = 0;
    float* out[H + 1];
    static_for<2, H>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        const int i = r0 + lane - a.c;
        if (i - m * floor_div<m>(i, a.c) == 0) begins |= 1u << m;
        out[m] = a.part + a.off[m] + (int64_t)rb * piece_rows(1 << a.shift, m) * partial_pitch(m, a.N, a.n_bt) + j0 / m;
    });
    constexpr uint32_t kAll = ~0u;

    Source src(a, lane, j0, r0);
    float V[H + 1][kV];
    static_for<2, H>([&](auto mc) {
#pragma unroll
        for (int v = 0; v < kV; ++v) V[decltype(mc)::value][v] = 0.0f;
    });
    const float sgn = src.sign();
    src.request(1, kAll);
#pragma unroll 1
    for (int r = r0; r < r1; ++r) {
        float G[H][kV];
        src.weights(r, G);
        uint32_t fl = (uint32_t)__builtin_amdgcn_readlane((int)begins, (r + 1 - r0) & 63);
        if (r + 1 < r1) src.request(0, fl);
        else fl = kAll;
        // suffix sums G_m = g_m + G_{m+1}, from the last plane down
#pragma unroll
        for (int m = H - 1; m >= 1; --m) {
#pragma unroll
            for (int v = 0; v < kV; ++v) G[m - 1][v] = G[m - 1][v] + G[m][v];
        }
        float* const dst = a.dfop + (int64_t)r * a.N + j0;
        if (!src.edge) {
            *reinterpret_cast<float4_a4*>(dst + kV * lane) =
                float4_a4{sgn * G[0][0], sgn * G[0][1], sgn * G[0][2], sgn * G[0][3]};
        } else {
#pragma unroll
            for (int v = 0; v < kV; ++v)
                if (j0 + kV * lane + v < a.N) dst[kV * lane + v] = sgn * G[0][v];
        }
        static_for<2, H>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
#pragma unroll
            for (int v = 0; v < kV; ++v) V[m][v] = V[m][v] + G[m - 1][v];
            if (fl & (1u << m)) {
#pragma unroll
                for (int v = 0; v < kV; ++v) V[m][v] = sgn * V[m][v];
                emit_targets<m>(V[m], row, j0, end, targets(m, a.N) + bt - j0 / m, lane, out[m]);
                out[m] += partial_pitch(m, a.N, a.n_bt);
#pragma unroll
                for (int v = 0; v < kV; ++v) V[m][v] = 0.0f;
            }
        });
    }
}

constexpr int bwd_occ(int H) { return H <= 8 ? 4 : 2; }

template <int H, bool NT>
__global__ __launch_bounds__(kGThreads, bwd_occ(H)) void k_bwd_tiles(BwdArgs a)
{
    __shared__ __align__(16) float lds[kGWaves * kGPitch];
    bwd_walk<H, PlaneSource<H, NT>>(a, lds);
}

template <typename TIn, int H>
__global__ __launch_bounds__(kGThreads, bwd_occ(H)) void k_lse_bwd_tiles(BwdArgs a)
{
    __shared__ __align__(16) float lds[kGWaves * kGPitch];
    bwd_walk<H, LseSource<TIn, H>>(a, lds);
}

// Pass 2: dFOP(a, b) += the partials covering (a, b), m = 2..H.  Rows a0 + y
// (those that some box meets), four consecutive bins per thread: per m and
// piece one vector load, and one element where a target of the four lies
// across two strips (at most one does).  What depends on the row alone is
// uniform.
template <int H, int S>
struct Reduce {
    static constexpr int R = 1 << S;              // rows of a piece
    const BwdArgs& a;
    int ar, b0;
    float add[4];

    // m = LO..HI, all their loads in flight together
    template <int LO, int HI>
    __device__ __forceinline__ void take()
    {
        constexpr int n = HI - LO + 1;
        float x[n][8], y[n][2];
        int vs[n];
        static_for<LO, HI>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            float(&xm)[8] = x[m - LO];
            float(&ym)[2] = y[m - LO];
#pragma unroll
            for (int v = 0; v < 8; ++v) xm[v] = 0.0f;
            ym[0] = ym[1] = 0.0f;
            vs[m - LO] = 4;
            const int i0 = a.c + m * (ar - a.c);
            const int first = max(i0, 0), last = min(i0 + m - 1, a.T - 1);
            if (first > last) return;
            const int nb = targets(m, a.N);
            if (b0 >= nb) return;
            // the strip of the four targets' last bin, and the one of them
            // that begins before it
            uint32_t o = 0;
            bool across = false;
            if constexpr (kTileBins % m != 0) {
                const int s = (m * (b0 + 4) - 1) / kTileBins, B = s * kTileBins;
                const int t = (int)((uint32_t)B / (uint32_t)m);
                across = m * b0 < B && t * m != B && B < a.N;
                vs[m - LO] = across ? t - b0 : 4;
                o = (uint32_t)(nb + s) * 4;
            }
            const int f = first / R, l = last / R;
            auto at = [&](int rb) {
                const int tr = ar - a.c - floor_div<m>(rb * R - a.c, a.c);
                return rows::scalar((gptr_t)(uintptr_t)(a.part + a.off[m] +
                                                        ((int64_t)rb * piece_rows(R, m) + tr) *
                                                            partial_pitch(m, a.N, a.n_bt)));
            };
            const gptr_t p = at(f);
            load4(p, xm);
            if (across) ym[0] = load1(p, o);
            if (l > f) {
                const gptr_t q = at(l);
                load4(q, xm + 4);
                if (across) ym[1] = load1(q, o);
                if constexpr (m > R + 1) {                // pieces lower than m
                    for (int rb = f + 1; rb < l; ++rb) {
                        const gptr_t z = at(rb);
                        float w[4];
                        load4(z, w);
#pragma unroll
                        for (int v = 0; v < 4; ++v) xm[v] += w[v];
                        if (across) ym[0] += load1(z, o);
                    }
                }
            }
        });
        static_for<LO, HI>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const float (&xm)[8] = x[m - LO];
            const float ys = y[m - LO][0] + y[m - LO][1];
            const int left = targets(m, a.N) - b0;        // the rest is not of this row
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float t = rows::opaque(xm[v]) + rows::opaque(xm[4 + v]);
                if constexpr (kTileBins % m != 0) t += v == vs[m - LO] ? ys : 0.0f;
                add[v] += v < left ? t : 0.0f;
            }
        });
    }
    __device__ __forceinline__ void load4(gptr_t p, float* x) const
    {
        uint32_t w[4];
        rows::load_words<4, 4>(p + (uint32_t)b0 * 4, w);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = __uint_as_float(w[v]);
    }
    __device__ static __forceinline__ float load1(gptr_t p, uint32_t o)
    {
        uint32_t w[1];
        rows::load_words<1, 4>(p + o, w);
        return __uint_as_float(w[0]);
    }
};

template <int H, int S>
__global__ __launch_bounds__(256, 4) void k_bwd_reduce(BwdArgs a, int a0, int n_rows)
{
    const int half = (a.N - 1) / 2 + 1;           // bins with an m = 2 box
    const int bl = 4 * (blockIdx.x * 256 + (int)threadIdx.x);
    if (bl >= half) return;
    for (int y = blockIdx.y; y < n_rows; y += gridDim.y) {
        const int b0 = rows::opaque(bl);          // nothing kept of every m from row to row
        Reduce<H, S> red{a, a0 + y, b0, {0.0f, 0.0f, 0.0f, 0.0f}};
        float* const d = a.dfop + (int64_t)(a0 + y) * a.N + b0;
        float4_a4 g = {0.0f, 0.0f, 0.0f, 0.0f};
        const bool whole = b0 + 4 <= a.N;
        if (whole) {
            g = *reinterpret_cast<const float4_a4*>(d);
        } else {
#pragma unroll
            for (int v = 0; v < 3; ++v)
                if (b0 + v < a.N) g[v] = d[v];
        }
        if constexpr (H <= 8) {
            red.template take<2, H>();
        } else {
            // in groups: registers
            red.template take<2, 6>();
            asm volatile("" ::: "memory");
            red.b0 = rows::opaque(b0);
            red.template take<7, (H < 11 ? H : 11)>();
            if constexpr (H > 11) {
                asm volatile("" ::: "memory");
                red.b0 = rows::opaque(b0);
                red.template take<12, H>();
            }
        }
        if (whole) {
            *reinterpret_cast<float4_a4*>(d) =
                float4_a4{g[0] + red.add[0], g[1] + red.add[1], g[2] + red.add[2], g[3] + red.add[3]};
        } else {
#pragma unroll
            for (int v = 0; v < 3; ++v)
                if (b0 + v < a.N) d[v] = g[v] + red.add[v];
        }
    }
}

// Log-sum-exp, level 1: block (k, i) reduces a contiguous chunk of plane k
// to a (max, sum of exp(x - max)) pair, x = HP / tau evaluated in fp64.
constexpr int kLseBlocks = 256;

__device__ __forceinline__ void lse_merge(double& M, float& S, double M2, float S2)
{
    if (S2 == 0.0f) return;
    if (S == 0.0f) { M = M2; S = S2; return; }
    if (M2 > M) { S = S * expf((float)(M - M2)) + S2; M = M2; }
    else S = S + S2 * expf((float)(M2 - M));
}

__global__ __launch_bounds__(256) void k_lse_part(const float* __restrict__ hp, int64_t plane, double inv_tau,
                                                  double* __restrict__ pm, float* __restrict__ ps)
{
    const int k = blockIdx.y;
    const int64_t chunk = (plane + gridDim.x - 1) / gridDim.x;
    const int64_t beg = blockIdx.x * chunk, end = min(plane, beg + chunk);
    const float* x = hp + (int64_t)k * plane;
    double M = 0.0;
    float S = 0.0f;
    for (int64_t e = beg + threadIdx.x; e < end; e += blockDim.x) {
        const double xd = (double)x[e] * inv_tau;
        if (S == 0.0f) { M = xd; S = 1.0f; }
        else if (xd > M) { S = S * expf((float)(M - xd)) + 1.0f; M = xd; }
        else S += expf((float)(xd - M));
    }
    __shared__ double sm[256];
    __shared__ float ss[256];
    sm[threadIdx.x] = M;
    ss[threadIdx.x] = S;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            double m1 = sm[threadIdx.x];
            float s1 = ss[threadIdx.x];
            lse_merge(m1, s1, sm[threadIdx.x + w], ss[threadIdx.x + w]);
            sm[threadIdx.x] = m1;
            ss[threadIdx.x] = s1;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        pm[(int64_t)k * gridDim.x + blockIdx.x] = sm[0];
        ps[(int64_t)k * gridDim.x + blockIdx.x] = ss[0];
    }
}

// Level 2: one thread per plane merges the block pairs in block order.
__global__ void k_lse_final(const double* __restrict__ pm, const float* __restrict__ ps, int H, int nblk,
                            double* __restrict__ lse)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= H) return;
    double M = 0.0;
    float S = 0.0f;
    for (int i = 0; i < nblk; ++i) lse_merge(M, S, pm[(int64_t)k * nblk + i], ps[(int64_t)k * nblk + i]);
    lse[k] = M + log((double)S);
}

// L = sum_k tau * lse[k-1], in k order (fp64).
__global__ void k_lse_loss(const double* __restrict__ lse, int H, double tau, double* __restrict__ loss)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double L = 0.0;
    for (int k = 0; k < H; ++k) L += tau * lse[k];
    *loss = L;
}

// Fused statistic, level 2: one block per plane.  The blocks' pairs (max
// m_b in storage units, sum s_b of exp((x - m_b) * cd)) are merged in fp64,
// cd = inv_scale / tau: first the largest m_b, then the sum of
// s_b * exp((m_b - M) * cd); each thread takes a fixed stride of blocks and
// the threads are combined by a fixed tree (deterministic).
// lse = M * cd + log(S).
constexpr int kLseFinalThreads = 256;

__global__ __launch_bounds__(kLseFinalThreads) void k_lse_fused_final(const float* __restrict__ part, int nblk, int H,
                                                                    double cd, double* __restrict__ lse)
{
    const int k = blockIdx.x;
    __shared__ double red[kLseFinalThreads];
    double m = -__builtin_inf();
    for (int b = threadIdx.x; b < nblk; b += kLseFinalThreads) {
        const double s2 = part[((int64_t)b * H + k) * 2 + 1];
        if (s2 != 0.0) m = fmax(m, (double)part[((int64_t)b * H + k) * 2]);
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kLseFinalThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    const double M = red[0];
    __syncthreads();
    double acc = 0.0;
    if (M != -__builtin_inf()) {
        for (int b = threadIdx.x; b < nblk; b += kLseFinalThreads) {
            const double s2 = part[((int64_t)b * H + k) * 2 + 1];
            if (s2 != 0.0) acc += s2 * exp(((double)part[((int64_t)b * H + k) * 2] - M) * cd);
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kLseFinalThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) lse[k] = M * cd + log(red[0]);
}

int grid_for(int64_t n, int threads, int cap)
{
    const int64_t b = (n + threads - 1) / threads;
    return (int)(b < cap ? (b < 1 ? 1 : b) : cap);
}

}  // namespace

// Rows of a piece (4, 8 or 16) from the plane's size alone: as many as leave
// enough pieces to even the load.  Tall pieces write fewer partial rows; the
// waves of the plain transpose stream, and want more of them (128 x 300001 at
// H = 8: 407 us with 16 rows, 351 with 8; the statistic's 132 and 152;
// 85 x 2^18: 203 / 196 / 203 us with 16 / 8 / 4 rows and 73 / 73 / 84).
int backward_shift(int T, int64_t N, bool planes)
{
    const int64_t n_bt = (N + kTileBins - 1) / kTileBins, least = planes ? 10000 : 8192;
    int shift = 4;
    while (shift > 2 && n_bt * ((T + (1 << shift) - 1) >> shift) < least) --shift;
    return shift;
}

int64_t backward_partial_floats(int T, int H, int64_t N, bool planes)
{
    const int shift = backward_shift(T, N, planes);
    const int64_t rows = (T + (1 << shift) - 1) >> shift, n_bt = (N + kTileBins - 1) / kTileBins;
    int64_t o = 0;
    for (int m = 2; m <= H; ++m) o += rows * piece_rows(1 << shift, m) * partial_pitch(m, (int)N, (int)n_bt);
    return o;
}

namespace {

bool bwd_args(BwdArgs& a, bool planes, const void* src, int64_t ld, int T, int64_t N, int H, float* dfop, float* part)
{
    a.src = src;
    a.ld = ld;
    a.T = T;
    a.c = T / 2;
    a.N = (int32_t)N;
    a.shift = backward_shift(T, N, planes);
    a.row_blocks = (T + (1 << a.shift) - 1) >> a.shift;
    a.n_bt = (int32_t)((N + kTileBins - 1) / kTileBins);
    a.dfop = dfop;
    a.part = part;
    int64_t o = 0;
    for (int m = 2; m <= kMaxH; ++m) {
        a.off[m] = o;
        o += (int64_t)a.row_blocks * piece_rows(1 << a.shift, m) * partial_pitch(m, a.N, a.n_bt);
    }
    return H >= 1 && H <= kMaxH && (int64_t)a.row_blocks * a.n_bt <= 0x7fffffff;
}

unsigned bwd_grid(const BwdArgs& a)
{
    const int64_t units = (int64_t)a.row_blocks * a.n_bt;
    return (unsigned)(8 * ((units + 8 * kGWaves - 1) / (8 * kGWaves) + 1));
}

// f(integral_constant<int, H>) for H = 1..kMaxH.
template <int HH, typename F>
void for_planes(int H, F&& f)
{
    if constexpr (HH <= kMaxH) {
        if (HH == H) f(std::integral_constant<int, HH>{});
        else for_planes<HH + 1>(H, f);
    }
}

template <int H>
hipError_t launch_bwd_reduce(const BwdArgs& a, hipStream_t s)
{
    if constexpr (H >= 2) {
        const int a0 = a.c - (a.c + 1) / 2, a1 = a.c + (a.T - 1 - a.c) / 2;   // rows with an m = 2 box
        const int n_rows = a1 - a0 + 1, half = (a.N - 1) / 2 + 1;
        const auto k = a.shift == 2 ? k_bwd_reduce<H, 2> : a.shift == 3 ? k_bwd_reduce<H, 3> : k_bwd_reduce<H, 4>;
        hipLaunchKernelGGL(k, dim3((half + 1023) / 1024, n_rows < 32768 ? n_rows : 32768), dim3(256), 0, s, a, a0, n_rows);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_backward(const float* g, float* dfop, float* part, int T, int64_t N, int H, hipStream_t s)
{
    BwdArgs a{};
    if (!bwd_args(a, true, g, 0, T, N, H, dfop, part)) return hipErrorInvalidValue;
    // Planes that the last-level cache (256 MB) cannot hold are read past it:
    // the tile pass of 85 x 2^18 (713 MB) in a training step 211 -> 173 us; of
    // planes that fit, it may hold what the caller has just written (101 x
    // 50000, 162 MB: a step with a product before it 298 us, 308 read past it).
    const bool nt = (int64_t)H * T * N * 4 > ((int64_t)256 << 20);
    hipError_t e = hipErrorInvalidValue;
    for_planes<1>(H, [&](auto hc) {
        constexpr int HH = decltype(hc)::value;
        const auto k = nt ? k_bwd_tiles<HH, true> : k_bwd_tiles<HH, false>;
        hipLaunchKernelGGL(k, dim3(bwd_grid(a)), dim3(kGThreads), 0, s, a);
        e = hipGetLastError();
        if (e == hipSuccess) e = launch_bwd_reduce<HH>(a, s);
    });
    return e;
}

hipError_t launch_lse_backward_fused(int dtype, const void* fop, int64_t ld, int T, int64_t N, int H, float inv_scale,
                                    double tau, const double* lse, const double* gscale, float* dfop, float* part,
                                    hipStream_t s)
{
    BwdArgs a{};
    if (!bwd_args(a, false, fop, ld, T, N, H, dfop, part)) return hipErrorInvalidValue;
    a.inv_scale = (double)inv_scale;
    a.tau = tau;
    a.c2 = (float)(1.4426950408889634 * (double)inv_scale / tau);   // log2(e) / (tau scale)
    a.lse = lse;
    a.gscale = gscale;
    hipError_t e = hipErrorInvalidValue;
    for_planes<1>(H, [&](auto hc) {
        constexpr int HH = decltype(hc)::value;
        const dim3 grid(bwd_grid(a)), block(kGThreads);
        switch (dtype) {
        case HS_DTYPE_F32: hipLaunchKernelGGL((k_lse_bwd_tiles<float, HH>), grid, block, 0, s, a); break;
        case HS_DTYPE_F16: hipLaunchKernelGGL((k_lse_bwd_tiles<_Float16, HH>), grid, block, 0, s, a); break;
        case HS_DTYPE_BF16: hipLaunchKernelGGL((k_lse_bwd_tiles<bf16_t, HH>), grid, block, 0, s, a); break;
        default: return;
        }
        e = hipGetLastError();
        if (e == hipSuccess) e = launch_bwd_reduce<HH>(a, s);
    });
    return e;
}

int64_t lse_part_bytes(int H) { return (int64_t)H * kLseBlocks * (8 + 4); }

hipError_t launch_lse_reduce(const float* hp, int64_t plane, int H, double tau, void* work, double* lse,
                             hipStream_t s)
{
    double* pm = static_cast<double*>(work);
    float* ps = reinterpret_cast<float*>(pm + (int64_t)H * kLseBlocks);
    hipLaunchKernelGGL(k_lse_part, dim3(kLseBlocks, H), dim3(256), 0, s, hp, plane, 1.0 / tau, pm, ps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lse_final, dim3(1), dim3(64), 0, s, pm, ps, H, kLseBlocks, lse);
    return hipGetLastError();
}

hipError_t launch_lse_fused_final(const float* part, int nblk, int H, double inv_scale, double tau,
                                  double* lse, hipStream_t s)
{
    hipLaunchKernelGGL(k_lse_fused_final, dim3(H), dim3(kLseFinalThreads), 0, s, part, nblk, H, inv_scale / tau, lse);
    return hipGetLastError();
}

hipError_t launch_lse_loss(const double* lse, int H, double tau, double* loss, hipStream_t s)
{
    hipLaunchKernelGGL(k_lse_loss, dim3(1), dim3(64), 0, s, lse, H, tau, loss);
    return hipGetLastError();
}


}  // namespace hsk
