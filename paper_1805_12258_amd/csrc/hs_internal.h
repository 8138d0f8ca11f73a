// Internal declarations of libhs: plan object, tile geometry, launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <vector>

#include "hs.h"

namespace hsk {

// Tile geometry of the fused kernels.  A tile is a block of at most
// kMaxTileRows template rows times kTileBins consecutive bins; each lane owns
// kV consecutive bins of one row at a time, and wave w of a block handles the
// tile rows w + q kWaves, q < kRowsPerWave.
constexpr int kLanes = 64;
constexpr int kV = 4;
constexpr int kTileBins = kV * kLanes;   // 256
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kLanes;
constexpr int kRowsPerWave = 4;
constexpr int kMaxTileRows = kWaves * kRowsPerWave;   // 32
constexpr int kMaxH = 16;
// LDS that a block of hs_sum and of the statistic reserves after its row table.
// The statistic's pairs take at most 1 KB of it; with the rest a plan's lds_bytes
// holds two blocks of five to thirteen planes to a compute unit (three would
// fit without), and the resident grid is the one the statistic's partial sums
// are formed over, whose order its last bits depend on.
constexpr int kTailBytes = 20656;

// Source words a tile needs per row of stretch factor m: the largest number
// of distinct floor(j/m) over kTileBins consecutive bins starting at a
// multiple of kTileBins (j0 mod m is then a multiple of gcd(kTileBins, m),
// which for a power-of-two tile width is the lowest set bit of m).
static_assert(kTailBytes >= kWaves * kMaxH * 2 * 4, "pairs of every wave and plane");
static_assert((kTileBins & (kTileBins - 1)) == 0, "tile width must be a power of two");
__host__ __device__ constexpr int stage_pitch(int m)
{
    return (m - (m & -m) + kTileBins - 1) / m + 1;
}

// Staging layout in LDS, fixed at compile time for tiles of up to
// kMaxTileRows rows.  Region m (m = 2..H) holds stage_rows(m) source rows of
// stage_row_words(m) words.  Rows are loaded in 16-byte pieces (LDS-DMA of
// four words per lane), so a row starts at the source word floor(j0/m)
// rounded down to a multiple of four; when m divides kTileBins / 4 that word
// is already aligned.
__host__ __device__ constexpr bool stage_aligned(int m) { return (kTileBins / 4) % m == 0; }
__host__ __device__ constexpr int stage_row_words(int m)
{
    return (stage_pitch(m) + (stage_aligned(m) ? 0 : 3) + 3) & ~3;
}
// Most distinct floor(i/m) over kMaxTileRows consecutive template indices.
__host__ __device__ constexpr int stage_rows(int m) { return (kMaxTileRows + m - 2) / m + 1; }
__host__ __device__ constexpr int stage_region_words(int m) { return stage_rows(m) * stage_row_words(m); }
__host__ __device__ constexpr int stage_offset(int m)
{
    int o = 0;
    for (int k = 2; k < m; ++k) o += stage_region_words(k);
    return o;
}
// Words of one staging buffer for H planes.
__host__ __device__ constexpr int stage_words(int H) { return stage_offset(H + 1); }

// LDS-DMA pieces: one wave instruction moves 64 lanes x 4 words.  Region m is
// covered by stage_chunks(m) pieces (the last one partly masked); pieces are
// numbered across regions and piece g is issued by wave g % kWaves.
constexpr int kDmaWords = kLanes * 4;
__host__ __device__ constexpr int stage_chunks(int m)
{
    return (stage_region_words(m) + kDmaWords - 1) / kDmaWords;
}
__host__ __device__ constexpr int stage_chunk_begin(int m)
{
    int o = 0;
    for (int k = 2; k < m; ++k) o += stage_chunks(k);
    return o;
}
__host__ __device__ constexpr int stage_total_chunks(int H) { return stage_chunk_begin(H + 1); }
__host__ __device__ constexpr int stage_chunk_m(int g)
{
    int m = 2;
    while (g >= stage_chunk_begin(m + 1)) ++m;
    return m;
}
__host__ __device__ constexpr int stage_slots(int H)
{
    return (stage_total_chunks(H) + kWaves - 1) / kWaves;
}
// Registers holding a wave's piece offsets (at least one, for H = 1).
__host__ __device__ constexpr int stage_slot_regs(int H) { return stage_slots(H) > 0 ? stage_slots(H) : 1; }

// Raw staging of 16-bit FOPs: the same source rectangles as 16-bit halves,
// loaded by the same 16-byte pieces (8 halves per lane) and converted to the
// fp32 layout above inside LDS.  A raw row starts at floor(j0/m) rounded down
// to 8 halves, i.e. (blo & 4) halves before the fp32 row, and holds the fp32
// row's words after that shift.
__host__ __device__ constexpr int raw_row_halves(int m)
{
    return (stage_row_words(m) + (stage_aligned(m) ? 0 : 4) + 7) & ~7;
}
__host__ __device__ constexpr int raw_region_halves(int m) { return stage_rows(m) * raw_row_halves(m); }
__host__ __device__ constexpr int raw_offset(int m)
{
    int o = 0;
    for (int k = 2; k < m; ++k) o += raw_region_halves(k);
    return o;
}
// Halves of one raw staging buffer for H planes.
__host__ __device__ constexpr int raw_halves(int H) { return raw_offset(H + 1); }
constexpr int kDmaHalves = kLanes * 8;
__host__ __device__ constexpr int raw_chunks(int m) { return (raw_region_halves(m) + kDmaHalves - 1) / kDmaHalves; }
__host__ __device__ constexpr int raw_chunk_begin(int m)
{
    int o = 0;
    for (int k = 2; k < m; ++k) o += raw_chunks(k);
    return o;
}
__host__ __device__ constexpr int raw_total_chunks(int H) { return raw_chunk_begin(H + 1); }
__host__ __device__ constexpr int raw_chunk_m(int g)
{
    int m = 2;
    while (g >= raw_chunk_begin(m + 1)) ++m;
    return m;
}
__host__ __device__ constexpr int raw_slots(int H) { return (raw_total_chunks(H) + kWaves - 1) / kWaves; }
// Piece slots of the storage type: raw pieces for 16-bit storage.
__host__ __device__ constexpr int dma_slots(int H, int elem_bytes)
{
    return elem_bytes == 4 ? stage_slots(H) : raw_slots(H);
}
__host__ __device__ constexpr int dma_slot_regs(int H, int elem_bytes)
{
    return dma_slots(H, elem_bytes) > 0 ? dma_slots(H, elem_bytes) : 1;
}

// Row table of a tile: per tile row, the staging offsets of stretch factors
// 2..H (padded to 4 words), then H words (padded to 4) that hold zero.
__host__ __device__ constexpr int row_table_thr_offset(int H) { return ((H - 1) + 3) & ~3; }
__host__ __device__ constexpr int row_table_stride(int H)
{
    return row_table_thr_offset(H) + ((H + 3) & ~3);
}

// The row table covers all T rows (and is built once per launch) when it
// takes at most this many bytes; otherwise it covers one tile's rows.
constexpr int kWholeTableBytes = 12 * 1024;
__host__ __device__ constexpr bool table_whole(int T, int H)
{
    return T * row_table_stride(H) * 4 <= kWholeTableBytes;
}

// LDS bytes after the two staging buffers: the row table (two per-tile
// copies unless it covers the whole plane) and the tail.
__host__ __device__ constexpr int smem_tail_bytes(int T, int R, int H)
{
    return (table_whole(T, H) ? T : 2 * R) * row_table_stride(H) * 4 +
           kTailBytes;
}

__host__ __device__ inline int64_t floordiv(int64_t a, int64_t b)
{
    int64_t q = a / b;
    return (q * b > a) ? q - 1 : q;
}

__host__ __device__ inline int floordiv32(int a, int b)
{
    int q = a / b;
    return (q * b > a) ? q - 1 : q;
}

// Arguments of one fused launch over one FOP (or one FOP of a batch).
struct TileArgs {
    const void* fop;
    int64_t ld;
    int64_t N;              // bins
    int32_t T;              // rows
    int32_t c;              // centre row: row r holds template index r - c
    int32_t R;              // rows per tile
    int32_t row_blocks;     // tiles across the rows
    float scale;            // stored = power * scale
    float inv_scale;        // applied when a stored value is converted to fp32
    int32_t table_whole;          // row table covers all T rows (built once)
    // materialised planes
    float* hp;              // [H][T][N]
    // Full-tile schedule: sched[0..8] are the offsets of eight lists in the
    // entries that follow, each entry (rb << 24) | bt.  Block b walks list
    // b % 8 with a stride of the number of blocks that share it.  Null: every
    // block takes a contiguous chunk of the row-block-major numbering.
    const uint32_t* sched;
    // fused log-sum-exp: per block and plane the pair (max, sum of
    // exp2((x - max) * lse_c)) of the block's values x in storage units
    float* lse_part;        // [gridDim.x][H][2]
    float lse_c;            // inv_scale * log2(e) / tau
};

// Arguments of the detection kernels (hs_rows.h), for one FOP
// (n_fops == 0: fop, ld, N, out, cap, counts) or a batch (n_fops >= 1: the
// per-FOP device arrays; out, counts are the bases).
struct WalkArgs {
    const void* fop;
    int64_t ld;
    int32_t N;
    int32_t n_fops;
    const void* const* fops;      // [n_fops] device
    const int64_t* lds;           // [n_fops] device
    const int64_t* n_chans;       // [n_fops] device (plan table)
    const int64_t* out_offsets;   // [n_fops] device
    const int64_t* caps;          // [n_fops] device
    int32_t T, c;                 // rows; row r holds template index r - c
    float scale, inv_scale;
    const float* ta;              // [H][T] unscaled
    hs_cand* out;
    int64_t cap;
    unsigned long long* counts;   // [H+1] (batch: [n_fops][H+1])
    int32_t s_row, s_bin;
    const uint32_t* ent;          // schedule entries: strips of 64 V bins
    const int32_t* seg;           // [n_seg][4]: FOP, first entry, first index, end index
    int32_t xseg[9];              // batch: segments of XCD x are [xseg[x], xseg[x+1])
    int32_t xfirst[8], xcount[8]; // single FOP: first entry and number of each XCD's strips
    int32_t lists;                // 8: a list per XCD; 1: one list that all XCDs take from
    int64_t units_per_list;       // strips of the longest list
    int32_t run;                  // units a wave takes one after another (set by the launcher)
    int32_t pieces;               // runs each half of a strip's rows is cut into (set by the launcher)
    int32_t lim_rows, lim_bins;   // batch: a FOP whose (ld * lim_rows + lim_bins) elements take
                                  // 2^32 bytes or more is rejected
};

enum Mode { kModeDetect = 0, kModeSum = 1, kModeLse = 2 };

// Fused log-sum-exp: most blocks one launch may use (the partial pairs of
// the workspace are sized for it).
constexpr int kLseMaxBlocks = 4096;

// Static device scratch of the allocation-free entry points: the fused
// statistic's per-block pairs at its largest grid and plane count.
constexpr size_t kNoAllocScratchBytes = (size_t)kLseMaxBlocks * kMaxH * 2 * sizeof(float);
// Address of this GPU's copy (looked up once per device).
hipError_t noalloc_scratch(void** ptr);

// LDS bytes of the fused kernel: fp32 storage double-buffers the fp32
// staging; 16-bit storage double-buffers the raw staging and converts into
// one fp32 staging buffer.
__host__ __device__ constexpr int fused_stage_bytes(int H, int elem_bytes)
{
    return elem_bytes == 4 ? 2 * stage_words(H) * 4 : stage_words(H) * 4 + 2 * ((raw_halves(H) * 2 + 15) & ~15);
}
int fused_lds_bytes(int T, int R, int H, int mode, int elem_bytes);

hipError_t launch_fused(int mode, int dtype, int H, const TileArgs& a, int64_t n_tiles,
                        int grid, int lds_bytes, hipStream_t s);
hipError_t launch_tiles(int dtype, int H, const WalkArgs& a, int grid, hipStream_t s);
hipError_t launch_stream_read(const void* src, int64_t bytes, float* sink, int grid, hipStream_t s);
hipError_t launch_zero_i64(int64_t* p, int64_t n, hipStream_t s);

// Bounded per-plane selection (policies of hs_select, n_cand <= kSelLdsCand).
constexpr int kSelLdsCand = 1024;
hipError_t select_bounded(const uint64_t* cand, int64_t n, int H, int s_bin, int s_k, int policy, int n_cand,
                          uint64_t* out, int64_t* out_counts, void* work, hipStream_t s);
size_t select_bounded_workspace(int64_t n, int H, int n_cand);

// Fractional mapping (HP_k = sum_{m<=k} FOP(floor(m i/k), floor(m j/k))):
// planes (hp) or detection (ta, out, cap, counts), single FOP, N <= 2^24.
constexpr int64_t kFracMaxBins = (int64_t)1 << 24;
struct FracArgs {
    const void* fop;
    int64_t ld;
    int32_t T, c, N, H;
    float scale, inv_scale;
    const float* ta;
    float* hp;
    hs_cand* out;
    int64_t cap;
    unsigned long long* counts;
    int32_t s_row, s_bin;
    // set by launch_frac: units of the work (strips x pieces of `rows` rows x
    // chains)
    int64_t units;
    int32_t pieces, rows, groups;
};
hipError_t launch_frac(int dtype, bool detect, const FracArgs& a, hipStream_t s);

// Strip-walk detection (hs_walk_*.hip): whether a plane takes it (at least
// two rows, thresholds of at most 16 KB), which bins-per-lane values V it is
// built for (strips of 64 V bins), and the launcher (grid <= 0: resident
// grid).
bool walk_supported(int T, int H);
bool walk_v_ok(int V);
hipError_t launch_walk(int dtype, int H, int V, const WalkArgs& a, int grid, hipStream_t s);

// Transpose of the plane map and the log-sum-exp statistic (hs_grad.hip).
// `part` holds backward_partial_floats(T, H, N, planes) floats (planes: of
// launch_backward, else of the statistic's).
int64_t backward_partial_floats(int T, int H, int64_t N, bool planes);
// The statistic's backward, its weights formed in the transpose's first pass.
hipError_t launch_lse_backward_fused(int dtype, const void* fop, int64_t ld, int T, int64_t N, int H, float inv_scale,
                                    double tau, const double* lse, const double* gscale, float* dfop, float* part,
                                    hipStream_t s);
hipError_t launch_backward(const float* g, float* dfop, float* part, int T, int64_t N, int H, hipStream_t s);
int64_t lse_part_bytes(int H);
hipError_t launch_lse_reduce(const float* hp, int64_t plane, int H, double tau, void* work, double* lse,
                             hipStream_t s);
hipError_t launch_lse_fused_final(const float* part, int nblk, int H, double inv_scale, double tau,
                                  double* lse, hipStream_t s);
hipError_t launch_lse_loss(const double* lse, int H, double tau, double* loss, hipStream_t s);
// Canonical candidate order (hs_sort.hip).
hipError_t sort_workspace(int64_t n, size_t* bytes);
hipError_t sort_candidates(uint64_t* cand, int64_t n, void* work, hipStream_t s);

}  // namespace hsk

struct hs_plan {
    int64_t T = 0;
    int64_t N = 0;          // single FOP: bins; batched: maximum bins
    int H = 0;
    int dtype = 0;
    float scale = 1.0f;
    int n_fops = 0;
    int mapping = HS_MAP_PAPER;
    std::vector<int64_t> n_chans;
    int s_row = 0, s_k = 0, s_bin = 0;
    int tile_rows = 0, row_blocks = 0;
    int lds_bytes = 0;
    int64_t tiles_total = 0;
    int persistent_blocks = 0;

    std::vector<uint32_t> sched;         // single FOP: full-tile schedule (empty: chunks)

    // Detection units and the tile schedule, host copy laid out as the device
    // buffer (offsets in bytes), copied once per device.
    bool walk = false;                   // the strip walk detects
    int walk_v = 4;                      // bins per lane (strips of 64 walk_v bins)
    std::vector<unsigned char> tab;
    size_t off_seg = 0, off_nchan = 0, off_ent = 0, off_sched = 0;
    int lists = 8;                       // strip lists: one per XCD, or one for all
    int64_t walk_units = 0;              // strips of the longest list
    int32_t xseg[9] = {0};               // batch: first segment of each XCD's
    int32_t xfirst[8] = {0}, xcount[8] = {0};   // single FOP: each XCD's strips

    // Device copies of `tab`, made on first use per device.
    mutable std::mutex mu;
    mutable unsigned char* d_tab[64] = {nullptr};
};
