// Host side of libhs: plan creation (shape checks, candidate-word widths,
// tile geometry), argument validation and kernel dispatch.  Every entry point
// returns an hs_status and catches C++ exceptions before they reach the ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <new>

#include "hs_internal.h"

namespace hsk {
// SingleHP baseline (hs_singlehp.hip)
hipError_t launch_singlehp(const float* fop, int64_t ld, int T, int N, int H, const float* ta, hs_cand* out,
                           int64_t cap, unsigned long long* counts, int s_row, int s_bin, float* work,
                           bool single_launch, hipStream_t s);
// Per-plane capped lists (hs_select.hip)
hipError_t select_workspace(int64_t n, int end_bit, size_t* bytes);
hipError_t select_top(const uint64_t* cand, int64_t n, int H, int s_bin, int s_k, int n_cand, uint64_t* out,
                      int64_t* out_counts, void* work, hipStream_t s);
}  // namespace hsk

namespace {

int ceil_log2(int64_t x)
{
    int s = 0;
    while (((int64_t)1 << s) < x) ++s;
    return s;
}

bool is_pow2_scale(float s)
{
    if (!(s > 0.0f) || !std::isfinite(s)) return false;
    int e = 0;
    return std::frexp(s, &e) == 0.5f;
}

int elem_bytes(int dtype) { return dtype == HS_DTYPE_F32 ? 4 : 2; }
int ld_align(int dtype) { return dtype == HS_DTYPE_F32 ? 4 : 8; }

// Largest LDS footprint the planner gives one block, so that two blocks fit
// in the 160 KiB of a gfx950 compute unit.
constexpr int kLdsBudget = 80 * 1024;

hs_status from_hip(hipError_t e) { return e == hipSuccess ? HS_OK : HS_ERR_HIP; }

bool fop_ok(const hs_plan* p, const void* fop, int64_t ld, int64_t N)
{
    if (!fop || ld < N) return false;
    if (reinterpret_cast<uintptr_t>(fop) & 15) return false;
    // the staging addresses source words by 32-bit byte offsets within the
    // source rows of one stretch factor (at most stage_rows(2) rows)
    if ((ld * hsk::stage_rows(2) + hsk::kTileBins) * elem_bytes(p->dtype) >= ((int64_t)1 << 32))
        return false;
    return ld % ld_align(p->dtype) == 0;
}

// Strip order of the detection kernels for one FOP of n_strips strips (the
// kernel side is described in hs_walk_impl.h).  Strip x >= 8 lies in
// octave L = floor(log2 x) at position (x - 2^L) / 2^L; its list is the three
// bits after the leading one, and dividing x by 2, 4 or 8 keeps both the list
// and the position scaled to the top octave.  Strips are ordered by that
// position, then by octave (x/8, x/4, x/2 just before x), then by index.
// lists == 8: one list per XCD; lists == 1: one list of all strips.
// The order is that of walking the binary tree in which x has the children
// 2x and 2x + 1, each strip followed by all it is an ancestor of, from the
// eight roots 8 .. 15 (list 1: the roots' trees advance together).
std::vector<std::vector<uint32_t>> walk_strip_lists(int64_t n_strips, int lists, bool linear = false)
{
    std::vector<std::vector<uint32_t>> out(lists);
    if (n_strips < 1) return out;
    for (auto& l : out) l.reserve((size_t)(n_strips / lists + n_strips / 16 + 2));
    if (linear) {
        // increasing strip order, dealt to the lists in turn
        for (int64_t x = 0; x < n_strips; ++x) out[x % lists].push_back((uint32_t)x);
        return out;
    }
    for (int64_t x = 0; x < n_strips && x < 8; ++x) out[lists == 8 ? x : 0].push_back((uint32_t)x);
    int top = 3;
    while (((int64_t)2 << top) <= n_strips - 1) ++top;      // octave of the last strip
    // positions p of the top octave's sub-ranges in order; the strips at
    // position p are those of the octaves whose step divides it
    for (int64_t p = 0; p < ((int64_t)1 << (top - 3)); ++p) {
        const int lo = p == 0 ? 3 : top - __builtin_ctzll((uint64_t)p);
        for (int k = 0; k < 8; ++k)
            for (int L = lo < 3 ? 3 : lo; L <= top; ++L) {
                const int64_t x = ((int64_t)1 << L) + ((int64_t)k << (L - 3)) + (p >> (top - L));
                if (x < n_strips) out[lists == 8 ? k : 0].push_back((uint32_t)x);
            }
    }
    return out;
}

// Full-tile schedule of a single-FOP plan (the kernel side is described in
// hs_fused_impl.h).  Bin tile x >= 8 lies in octave L = floor(log2 x); list
// k holds the tiles whose bits L-1..L-3 equal k (tiles 0..7 go to list x),
// ordered by their position inside that sub-range scaled to the top octave,
// then by L (so x/2, x/4, x/8 come just before x), then by row block.
// Layout: nine list offsets, then the entries (rb << 24) | x.  Empty when
// the fields do not fit.
// `lists` are those of n_full tiles or of one more (walk_strip_lists; the order
// of the tiles that they share is the same).
std::vector<uint32_t> build_schedule(const std::vector<std::vector<uint32_t>>& lists, int64_t n_full, int row_blocks)
{
    std::vector<uint32_t> out;
    if (n_full < 1 || row_blocks < 1 || row_blocks > 255 || n_full >= ((int64_t)1 << 24)) return out;
    out.reserve(9 + (size_t)n_full * row_blocks);
    out.assign(9, 0);
    for (int k = 0; k < 8; ++k) {
        for (uint32_t x : lists[k]) {
            if (x >= n_full) continue;
            for (int rb = 0; rb < row_blocks; ++rb) out.push_back(((uint32_t)rb << 24) | x);
        }
        out[k + 1] = (uint32_t)(out.size() - 9);
    }
    return out;
}

// A run of `count` units of FOP f from entry `first` of the unit list.
struct Run {
    int32_t f;
    int64_t first, count;
};

// The runs dealt to each XCD, evened out: XCDs with more than an eighth of
// the units hand their last ones to those with fewer.  (Bin counts that are
// no power of two leave the octave lists uneven, and few FOPs the batch's.)
void even_runs(std::vector<Run> (&on)[8])
{
    int64_t total = 0, has[8];
    for (int x = 0; x < 8; ++x) {
        has[x] = 0;
        for (const Run& r : on[x]) has[x] += r.count;
        total += has[x];
    }
    const int64_t quota = (total + 7) / 8;
    std::vector<Run> pool;
    for (int x = 0; x < 8; ++x) {
        while (has[x] > quota) {
            Run& r = on[x].back();
            const int64_t n = std::min(r.count, has[x] - quota);
            pool.push_back({r.f, r.first + r.count - n, n});
            r.count -= n;
            has[x] -= n;
            if (r.count == 0) on[x].pop_back();
        }
    }
    size_t q = 0;
    for (int x = 0; x < 8 && q < pool.size(); ++x) {
        while (has[x] < quota && q < pool.size()) {
            Run& r = pool[q];
            const int64_t n = std::min(r.count, quota - has[x]);
            on[x].push_back({r.f, r.first, n});
            r.first += n;
            r.count -= n;
            has[x] += n;
            if (r.count == 0) ++q;
        }
    }
}

// Detection units of a plan: the strips of every FOP (64 V bins; 256-bin
// tiles for the tile kernel).  A single FOP spreads its strips over eight XCD
// lists, a batch puts each FOP whole on one XCD (longest first onto the least
// loaded XCD); the lists are then evened out.
// Device layout: seg [n_seg][4] i32 | n_chans [n_fops] i64 | entries u32 | tile
// schedule u32 (one buffer, so that a plan takes one allocation and one copy).
// `tiles`: the lists of the 256-bin tiles of a single FOP, where they are those
// of the strips.
void build_units(hs_plan* p, bool walk, bool linear, const std::vector<std::vector<uint32_t>>& tiles)
{
    const int64_t sb = walk ? 64 * (int64_t)p->walk_v : hsk::kTileBins;
    std::vector<uint32_t> ent;
    auto add_units = [&](const std::vector<uint32_t>& strips) {
        const size_t first = ent.size();
        ent.insert(ent.end(), strips.begin(), strips.end());
        return std::make_pair((int64_t)first, (int64_t)strips.size());
    };
    std::vector<Run> on[8];
    std::vector<int64_t> nchan;
    if (p->n_fops == 0) {
        const bool same = !linear && sb == hsk::kTileBins && !tiles.empty();
        const auto own = same ? std::vector<std::vector<uint32_t>>() : walk_strip_lists((p->N + sb - 1) / sb, 8, linear);
        const auto& lists = same ? tiles : own;
        ent.reserve((size_t)((p->N + sb - 1) / sb));
        for (int x = 0; x < 8; ++x) {
            const auto r = add_units(lists[x]);
            if (r.second > 0) on[x].push_back({0, r.first, r.second});
        }
    } else {
        // one unit list per distinct number of strips
        std::map<int64_t, std::pair<int64_t, int64_t>> by_strips;     // -> (first, count)
        std::vector<std::pair<int64_t, int64_t>> fl(p->n_fops);
        for (int f = 0; f < p->n_fops; ++f) {
            const int64_t n = (p->n_chans[f] + sb - 1) / sb;
            auto it = by_strips.find(n);
            if (it == by_strips.end()) it = by_strips.emplace(n, add_units(walk_strip_lists(n, 1, linear)[0])).first;
            fl[f] = it->second;
        }
        // whole FOPs to XCDs: longest first onto the least loaded
        std::vector<int> order(p->n_fops);
        for (int f = 0; f < p->n_fops; ++f) order[f] = f;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return fl[a].second > fl[b].second; });
        std::vector<int> to(p->n_fops);
        int64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int f : order) {
            int best = 0;
            for (int x = 1; x < 8; ++x)
                if (load[x] < load[best]) best = x;
            to[f] = best;
            load[best] += fl[f].second;
        }
        for (int f = 0; f < p->n_fops; ++f)
            if (fl[f].second > 0) on[to[f]].push_back({(int32_t)f, fl[f].first, fl[f].second});
        nchan = p->n_chans;
    }
    even_runs(on);
    // Few strips of many rows: lists of whole strips cannot be even (a plane of
    // 256 bins would be walked by one XCD), so where the longest is more than
    // an eighth above the mean, and has more pieces of three rows than an XCD
    // has waves to walk them at once (512 to 768), the waves of all XCDs share
    // one list.  2^20 x 200 bins 1830 us by one XCD, 270 so; 85 x 1000, whose
    // pieces all fit, 18 us by lists, 19 by one.
    int64_t total = 0, longest = 0;
    for (const auto& l : on) {
        int64_t n = 0;
        for (const Run& r : l) n += r.count;
        total += n;
        longest = std::max(longest, n);
    }
    p->lists = 8 * longest * 8 > 9 * total && longest * p->T > 3 * 512 ? 1 : 8;
    if (p->lists == 1)
        for (int x = 1; x < 8; ++x) {
            on[0].insert(on[0].end(), on[x].begin(), on[x].end());
            on[x].clear();
        }
    if (p->n_fops == 0) {
        // one contiguous run of entries per XCD
        std::vector<uint32_t> all;
        all.reserve(ent.size());
        for (int x = 0; x < 8; ++x) {
            const size_t first = all.size();
            for (const Run& r : on[x]) all.insert(all.end(), ent.begin() + r.first, ent.begin() + r.first + r.count);
            p->xfirst[x] = (int32_t)first;
            p->xcount[x] = (int32_t)(all.size() - first);
            on[x].clear();
            if (all.size() > first) on[x].push_back({0, (int64_t)first, (int64_t)(all.size() - first)});
        }
        ent.swap(all);
    }

    std::vector<int32_t> seg;   // 4 per segment: FOP, first entry, first index, end index
    p->walk_units = 0;
    for (int x = 0; x < 8; ++x) {
        p->xseg[x] = (int32_t)(seg.size() / 4);
        int64_t pre = 0;
        for (const Run& r : on[x]) {
            seg.insert(seg.end(), {r.f, (int32_t)r.first, (int32_t)pre, (int32_t)(pre + r.count)});
            pre += r.count;
        }
        p->walk_units = std::max(p->walk_units, pre);
    }
    p->xseg[8] = (int32_t)(seg.size() / 4);

    auto align = [](size_t x) { return (x + 255) & ~(size_t)255; };
    p->off_seg = 0;
    p->off_nchan = align(p->off_seg + seg.size() * 4);
    p->off_ent = align(p->off_nchan + nchan.size() * 8);
    p->off_sched = align(p->off_ent + ent.size() * 4);
    p->tab.assign(p->off_sched + p->sched.size() * 4, 0);
    auto put = [&](size_t off, const auto& v) {
        if (!v.empty()) std::memcpy(p->tab.data() + off, v.data(), v.size() * sizeof(v[0]));
    };
    put(p->off_seg, seg);
    put(p->off_nchan, nchan);
    put(p->off_ent, ent);
    put(p->off_sched, p->sched);
    p->walk = walk;
}

// Device copies of a plan's tables on one device.
struct DevTabs {
    const unsigned char* walk = nullptr;   // detection units
    const uint32_t* sched = nullptr;       // full-tile schedule (null: contiguous chunks)
};

DevTabs tables_at(const hs_plan* p, const unsigned char* tab)
{
    DevTabs t;
    t.walk = tab;
    if (tab && !p->sched.empty()) t.sched = reinterpret_cast<const uint32_t*>(tab + p->off_sched);
    return t;
}

hs_status copy_to_device(const void* src, size_t bytes, void** dst)
{
    void* d = nullptr;
    if (hipMalloc(&d, bytes) != hipSuccess) return HS_ERR_NOMEM;
    if (hipMemcpy(d, src, bytes, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(d);
        return HS_ERR_HIP;
    }
    *dst = d;
    return HS_OK;
}

// Every table the plan has, on the current device: all are copied together
// (synchronously) by the first call on a device that is not under stream
// capture, or by hs_plan_upload.  A call under capture on a device that has
// no copy yet gets HS_ERR_INVALID, since a copy cannot be made inside a
// graph; so does a stream of another device than the current one (the
// tables are per device).
hs_status device_tables(const hs_plan* p, hipStream_t stream, DevTabs* t)
{
    *t = DevTabs{};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return HS_ERR_HIP;
    if (stream) {
        hipDevice_t sd = 0;
        if (hipStreamGetDevice(stream, &sd) != hipSuccess || (int)sd != dev) return HS_ERR_INVALID;
    }
    std::lock_guard<std::mutex> g(p->mu);
    if (!p->tab.empty() && !p->d_tab[dev]) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &cs) != hipSuccess) return HS_ERR_HIP;
        if (cs != hipStreamCaptureStatusNone) return HS_ERR_INVALID;
        void* d = nullptr;
        const hs_status st = copy_to_device(p->tab.data(), p->tab.size(), &d);
        if (st != HS_OK) return st;
        p->d_tab[dev] = static_cast<unsigned char*>(d);
    }
    *t = tables_at(p, p->d_tab[dev]);
    return HS_OK;
}

// The tables already on the current device, copying nothing (what is not
// there yet is null: the tile kernels then take contiguous chunks, with the
// same results).  HS_ERR_INVALID for a stream of another device.
hs_status device_tables_present(const hs_plan* p, hipStream_t stream, DevTabs* t)
{
    *t = DevTabs{};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return HS_ERR_HIP;
    if (stream) {
        hipDevice_t sd = 0;
        if (hipStreamGetDevice(stream, &sd) != hipSuccess || (int)sd != dev) return HS_ERR_INVALID;
    }
    std::lock_guard<std::mutex> g(p->mu);
    *t = tables_at(p, p->d_tab[dev]);
    return HS_OK;
}

hsk::WalkArgs walk_args(const hs_plan* p, const unsigned char* tab)
{
    hsk::WalkArgs a{};
    a.T = (int32_t)p->T;
    a.c = (int32_t)(p->T / 2);
    a.scale = p->scale;
    a.inv_scale = 1.0f / p->scale;
    a.s_row = p->s_row;
    a.s_bin = p->s_bin;
    std::memcpy(a.xseg, p->xseg, sizeof(a.xseg));
    a.lists = p->lists;
    a.units_per_list = p->walk_units;
    std::memcpy(a.xfirst, p->xfirst, sizeof(a.xfirst));
    std::memcpy(a.xcount, p->xcount, sizeof(a.xcount));
    a.lim_rows = p->walk ? (int32_t)p->T : hsk::stage_rows(2);
    a.lim_bins = p->walk ? 0 : hsk::kTileBins;
    a.seg = reinterpret_cast<const int32_t*>(tab + p->off_seg);
    a.n_chans = reinterpret_cast<const int64_t*>(tab + p->off_nchan);
    a.ent = reinterpret_cast<const uint32_t*>(tab + p->off_ent);
    return a;
}

// The plan's detection kernel.
hipError_t launch_detect(const hs_plan* p, const hsk::WalkArgs& a, hipStream_t s)
{
    return p->walk ? hsk::launch_walk(p->dtype, p->H, p->walk_v, a, p->persistent_blocks, s)
                   : hsk::launch_tiles(p->dtype, p->H, a, p->persistent_blocks, s);
}

hsk::FracArgs frac_args(const hs_plan* p, const void* fop, int64_t ld)
{
    hsk::FracArgs a{};
    a.fop = fop;
    a.ld = ld;
    a.T = (int32_t)p->T;
    a.c = (int32_t)(p->T / 2);
    a.N = (int32_t)p->N;
    a.H = p->H;
    a.scale = p->scale;
    a.inv_scale = 1.0f / p->scale;
    a.s_row = p->s_row;
    a.s_bin = p->s_bin;
    return a;
}

hsk::TileArgs tile_args(const hs_plan* p, const void* fop, int64_t ld, const DevTabs& t)
{
    hsk::TileArgs a{};
    a.fop = fop;
    a.ld = ld;
    a.N = p->N;
    a.T = (int32_t)p->T;
    a.c = (int32_t)(p->T / 2);
    a.R = p->tile_rows;
    a.row_blocks = p->row_blocks;
    a.scale = p->scale;
    a.inv_scale = 1.0f / p->scale;
    a.table_whole = hsk::table_whole((int)p->T, p->H) ? 1 : 0;
    a.sched = t.sched;
    return a;
}

int64_t bin_tiles(int64_t n) { return (n + hsk::kTileBins - 1) / hsk::kTileBins; }

}  // namespace

extern "C" {

hs_status hs_plan_create(hs_plan** out, const hs_plan_desc* d)
{
    if (!out || !d) return HS_ERR_INVALID;
    *out = nullptr;
    try {
        if (d->n_temp < 1 || d->n_temp > (1 << 20)) return HS_ERR_INVALID;
        if (d->n_hp < 1 || d->n_hp > hsk::kMaxH) return HS_ERR_INVALID;
        if (d->dtype != HS_DTYPE_F32 && d->dtype != HS_DTYPE_F16 && d->dtype != HS_DTYPE_BF16)
            return HS_ERR_INVALID;
        const float scale = d->input_scale == 0.0f ? 1.0f : d->input_scale;
        if (!is_pow2_scale(scale)) return HS_ERR_INVALID;
        if (d->dtype == HS_DTYPE_F32 && scale != 1.0f) return HS_ERR_INVALID;
        if (d->n_fops < 0 || d->n_fops > 65535) return HS_ERR_INVALID;
        if (d->tile_rows < 0 || d->persistent_blocks < 0) return HS_ERR_INVALID;
        if (d->schedule < 0 || d->schedule > 4) return HS_ERR_INVALID;
        if (d->mapping != HS_MAP_PAPER && d->mapping != HS_MAP_FRACTIONAL) return HS_ERR_INVALID;
        if (d->bins_per_lane != 0 && !hsk::walk_v_ok(d->bins_per_lane)) return HS_ERR_INVALID;
        if (d->mapping == HS_MAP_FRACTIONAL && (d->n_fops != 0 || d->n_chan > hsk::kFracMaxBins))
            return HS_ERR_INVALID;

        hs_plan* p = new hs_plan();
        p->mapping = d->mapping;
        // bins per lane of the strip walk: eight for 16-bit storage up to
        // eight planes and for batches, else four.  us a call at 8 / 4 / 2:
        // 85 x 2^21 fp16, eight planes 131 / 141 / 254, four planes 85 / 109 /
        // 189; bf16 85 x 2^20 71 / 81 / 122; six FOPs of 85 x 2^20, fp32 at 16
        // planes 720 / 736 / 1164, fp16 at eight 358 / 439 / 753.  Where four is
        // the choice the two are alike (fp32 174 / 176; 16 planes, where a
        // strip of eight is walked as two halves, 249 / 253 fp32 and 247 / 247
        // fp16; 85 x 2^18 at 16 planes 53 / 47); small planes want more strips
        // (21 x 2^16 fp16 14.1 / 12.5)
        p->walk_v = d->bins_per_lane ? d->bins_per_lane
                                     : ((d->dtype != HS_DTYPE_F32 && d->n_hp <= 8) || d->n_fops > 0 ? 8 : 4);
        p->T = d->n_temp;
        p->H = d->n_hp;
        p->dtype = d->dtype;
        p->scale = scale;
        p->n_fops = d->n_fops;
        p->persistent_blocks = d->persistent_blocks;
        int64_t nmax = 0;
        if (d->n_fops == 0) {
            if (d->n_chan < 1 || d->n_chan > INT32_MAX) { delete p; return HS_ERR_INVALID; }
            nmax = d->n_chan;
        } else {
            if (!d->n_chans) { delete p; return HS_ERR_INVALID; }
            p->n_chans.assign(d->n_chans, d->n_chans + d->n_fops);
            for (int64_t n : p->n_chans) {
                if (n < 1 || n > INT32_MAX) { delete p; return HS_ERR_INVALID; }
                if (n > nmax) nmax = n;
            }
        }
        p->N = nmax;
        p->s_bin = ceil_log2(nmax);
        p->s_k = ceil_log2(p->H);
        const int s_r = ceil_log2(p->T);
        if (p->s_bin + p->s_k + s_r > 32) { delete p; return HS_ERR_INVALID; }
        p->s_row = p->s_bin + p->s_k;

        // Rows per tile: kMaxTileRows (the staging layout is sized for it;
        // the last row block may be shorter), or fewer on request.
        int R = (int)std::min<int64_t>(d->tile_rows > 0 ? d->tile_rows : hsk::kMaxTileRows, p->T);
        if (R > hsk::kMaxTileRows ||
            hsk::fused_lds_bytes((int)p->T, R, p->H, hsk::kModeDetect, elem_bytes(p->dtype)) > kLdsBudget) {
            delete p;
            return HS_ERR_UNSUPPORTED;
        }
        p->tile_rows = R;
        p->row_blocks = (int)((p->T + R - 1) / R);
        p->lds_bytes = hsk::fused_lds_bytes((int)p->T, R, p->H, hsk::kModeDetect, elem_bytes(p->dtype));

        // detection: one walk over rows (hs_rows.h) under two names.  The strip
        // walk takes walk_v bins per lane, the tile kernel four: the same
        // kernel where walk_v is four (fp32 85 x 2^21 176 us by either name),
        // so the choice matters for the 16-bit planes and batches above.
        // schedule 1 and 4 ask for the strip walk, 2 and 3 for the tile kernel;
        // 0 and 4, 2 deal strips to XCDs by octave position, 1 and 3 in
        // increasing order.  The tile kernels of the other calls use the XCD
        // tile schedule for 0, 2 and 4, contiguous chunks for 1 and 3.
        const bool walk_wins = p->dtype != HS_DTYPE_F32 || p->H > 8;
        const bool want_walk = d->schedule == 1 || d->schedule == 4 || (d->schedule == 0 && walk_wins);
        const bool paper = d->mapping == HS_MAP_PAPER;   // the fractional mapping has a kernel of its own
        const bool walk = paper && want_walk && hsk::walk_supported((int)p->T, p->H);

        std::vector<std::vector<uint32_t>> tiles;
        if (d->n_fops == 0) {
            p->tiles_total = p->row_blocks * bin_tiles(p->N);
            if (paper && (d->schedule == 0 || d->schedule == 2 || d->schedule == 4)) {
                tiles = walk_strip_lists(bin_tiles(p->N), 8);
                p->sched = build_schedule(tiles, p->N / hsk::kTileBins, p->row_blocks);
            }
        } else {
            int64_t acc = 0;
            for (int64_t n : p->n_chans) acc += p->row_blocks * bin_tiles(n);
            p->tiles_total = acc;
        }
        if (paper) build_units(p, walk, d->schedule == 1 || d->schedule == 3, tiles);
        *out = p;
        return HS_OK;
    } catch (const std::bad_alloc&) {
        return HS_ERR_NOMEM;
    } catch (...) {
        return HS_ERR_INVALID;
    }
}

hs_status hs_plan_destroy(hs_plan* p)
{
    if (!p) return HS_OK;
    int cur = -1;
    bool have_dev = hipGetDevice(&cur) == hipSuccess;
    for (int dev = 0; dev < 64; ++dev) {
        if (p->d_tab[dev]) {
            if (have_dev) (void)hipSetDevice(dev);
            (void)hipFree(p->d_tab[dev]);
        }
    }
    if (have_dev && cur >= 0) (void)hipSetDevice(cur);
    delete p;
    return HS_OK;
}

int64_t hs_plan_schedule(const hs_plan* p, uint32_t* words, int64_t capacity)
{
    if (!p) return -1;
    const int64_t n = (int64_t)p->sched.size();
    if (words && capacity > 0) std::memcpy(words, p->sched.data(), (size_t)std::min(n, capacity) * 4);
    return n;
}

hs_status hs_plan_upload(const hs_plan* p)
{
    if (!p) return HS_ERR_INVALID;
    try {
        DevTabs t;
        return device_tables(p, nullptr, &t);
    } catch (...) {
        return HS_ERR_HIP;
    }
}

hs_status hs_plan_info_get(const hs_plan* p, hs_plan_info* info)
{
    if (!p || !info) return HS_ERR_INVALID;
    std::memset(info, 0, sizeof(*info));
    info->n_temp = (int32_t)p->T;
    info->n_hp = p->H;
    info->dtype = p->dtype;
    info->n_fops = p->n_fops;
    info->n_chan_max = p->N;
    info->s_row = p->s_row;
    info->s_k = p->s_k;
    info->s_bin = p->s_bin;
    info->tile_bins = hsk::kTileBins;
    info->tile_rows = p->tile_rows;
    info->row_blocks = p->row_blocks;
    info->lds_bytes = p->lds_bytes;
    info->tiles_total = p->tiles_total;
    info->detector = p->mapping == HS_MAP_FRACTIONAL ? 2 : (p->walk ? 1 : 0);
    info->mapping = p->mapping;
    info->bins_per_lane = p->walk ? p->walk_v : 0;
    // distinct source rows of each stretch factor over the full column, and the
    // words one full-height tile at a 256-bin aligned position stages
    const int64_t c = p->T / 2;
    int64_t staged = 0;
    for (int m = 1; m <= p->H; ++m) {
        const int64_t rows = hsk::floordiv(p->T - 1 - c, m) - hsk::floordiv(-c, m) + 1;
        info->src_rows[m] = (int32_t)rows;
        if (m >= 2) staged += rows * ((hsk::kTileBins - 1) / m + 1);
    }
    info->staged_words = staged;
    return HS_OK;
}

hs_status hs_sum(const hs_plan* p, const void* fop, int64_t ld, float* hp, void* stream)
{
    if (!p || !hp || p->n_fops != 0) return HS_ERR_INVALID;
    if (!fop_ok(p, fop, ld, p->N)) return HS_ERR_INVALID;
    try {
        if (p->mapping == HS_MAP_FRACTIONAL) {
            hsk::FracArgs a = frac_args(p, fop, ld);
            a.hp = hp;
            return from_hip(hsk::launch_frac(p->dtype, false, a, (hipStream_t)stream));
        }
        DevTabs t;
        const hs_status st = device_tables(p, (hipStream_t)stream, &t);
        if (st != HS_OK) return st;
        hsk::TileArgs a = tile_args(p, fop, ld, t);
        a.hp = hp;
        return from_hip(hsk::launch_fused(hsk::kModeSum, p->dtype, p->H, a, p->tiles_total,
                                          p->persistent_blocks, p->lds_bytes,
                                          (hipStream_t)stream));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

hs_status hs_detect(const hs_plan* p, const void* fop, int64_t ld, const float* ta, hs_cand* out,
                    int64_t capacity, int64_t* counts, void* stream)
{
    if (!p || p->n_fops != 0 || !ta || !counts || capacity < 0) return HS_ERR_INVALID;
    if (capacity > 0 && !out) return HS_ERR_INVALID;
    if (!fop_ok(p, fop, ld, p->N)) return HS_ERR_INVALID;
    try {
        hipStream_t s = (hipStream_t)stream;
        DevTabs t;
        const hs_status st = device_tables(p, s, &t);
        if (st != HS_OK) return st;
        if (p->mapping == HS_MAP_FRACTIONAL) {
            if (hsk::launch_zero_i64(counts, p->H + 1, s) != hipSuccess) return HS_ERR_HIP;
            hsk::FracArgs a = frac_args(p, fop, ld);
            a.ta = ta;
            a.out = out;
            a.cap = capacity;
            a.counts = reinterpret_cast<unsigned long long*>(counts);
            if (hsk::launch_frac(p->dtype, true, a, s) != hipSuccess) return HS_ERR_HIP;
        } else {
            if (hsk::launch_zero_i64(counts, p->H + 1, s) != hipSuccess) return HS_ERR_HIP;
            hsk::WalkArgs a = walk_args(p, t.walk);
            a.fop = fop;
            a.ld = ld;
            a.N = (int32_t)p->N;
            a.n_fops = 0;
            a.ta = ta;
            a.out = out;
            a.cap = capacity;
            a.counts = reinterpret_cast<unsigned long long*>(counts);
            if (launch_detect(p, a, s) != hipSuccess) return HS_ERR_HIP;
        }
        return HS_OK;
    } catch (...) {
        return HS_ERR_HIP;
    }
}

size_t hs_select_workspace_bytes(const hs_plan* p, int64_t n)
{
    if (!p || n < 0) return 0;
    size_t bytes = 0;
    if (hsk::select_workspace(n, 32 + p->s_k, &bytes) != hipSuccess) return 0;
    return std::max(bytes, hsk::select_bounded_workspace(n, p->H, hsk::kSelLdsCand));
}

hs_status hs_select(const hs_plan* p, const hs_cand* cand, int64_t n, int32_t n_cand, int32_t policy, hs_cand* out,
                    int64_t* out_counts, void* work, void* stream)
{
    if (!p || n < 0 || n_cand < 1 || !out || !out_counts || !work) return HS_ERR_INVALID;
    if (policy != HS_SELECT_TOP && policy != HS_SELECT_LAST_ALG2 && policy != HS_SELECT_LAST_ALG1)
        return HS_ERR_INVALID;
    if (n > 0 && !cand) return HS_ERR_INVALID;
    try {
        const uint64_t* c = reinterpret_cast<const uint64_t*>(cand);
        uint64_t* o = reinterpret_cast<uint64_t*>(out);
        hipStream_t s = (hipStream_t)stream;
        if (n_cand <= hsk::kSelLdsCand && n <= (int64_t)UINT32_MAX)
            return from_hip(hsk::select_bounded(c, n, p->H, p->s_bin, p->s_k, policy, n_cand, o, out_counts, work, s));
        if (policy != HS_SELECT_TOP) return HS_ERR_UNSUPPORTED;
        return from_hip(hsk::select_top(c, n, p->H, p->s_bin, p->s_k, n_cand, o, out_counts, work, s));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

hs_status hs_select_top(const hs_plan* p, const hs_cand* cand, int64_t n, int32_t n_cand, hs_cand* out,
                        int64_t* out_counts, void* work, void* stream)
{
    return hs_select(p, cand, n, n_cand, HS_SELECT_TOP, out, out_counts, work, stream);
}

size_t hs_singlehp_workspace_bytes(const hs_plan* p)
{
    if (!p || p->n_fops != 0 || p->dtype != HS_DTYPE_F32) return 0;
    return 2 * (size_t)((p->T * p->N + 63) & ~(int64_t)63) * sizeof(float);
}

namespace {

hs_status singlehp(const hs_plan* p, const float* fop, int64_t ld, const float* ta, hs_cand* out, int64_t capacity,
                   int64_t* counts, void* work, bool single_launch, void* stream)
{
    if (!p || p->n_fops != 0 || !ta || !counts || !work || capacity < 0) return HS_ERR_INVALID;
    if (p->dtype != HS_DTYPE_F32 || p->mapping != HS_MAP_PAPER) return HS_ERR_UNSUPPORTED;
    if (capacity > 0 && !out) return HS_ERR_INVALID;
    if (!fop_ok(p, fop, ld, p->N)) return HS_ERR_INVALID;
    try {
        hipStream_t s = (hipStream_t)stream;
        hipError_t e = hsk::launch_zero_i64(counts, p->H + 1, s);
        if (e != hipSuccess) return HS_ERR_HIP;
        return from_hip(hsk::launch_singlehp(fop, ld, (int)p->T, (int)p->N, p->H, ta, out, capacity,
                                             reinterpret_cast<unsigned long long*>(counts), p->s_row, p->s_bin,
                                             static_cast<float*>(work), single_launch, s));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

}  // namespace

hs_status hs_detect_singlehp(const hs_plan* p, const float* fop, int64_t ld, const float* ta, hs_cand* out,
                             int64_t capacity, int64_t* counts, void* work, void* stream)
{
    return singlehp(p, fop, ld, ta, out, capacity, counts, work, false, stream);
}

hs_status hs_detect_singlehp_one(const hs_plan* p, const float* fop, int64_t ld, const float* ta, hs_cand* out,
                                 int64_t capacity, int64_t* counts, void* work, void* stream)
{
    return singlehp(p, fop, ld, ta, out, capacity, counts, work, true, stream);
}

hs_status hs_detect_batched(const hs_plan* p, const void* const* fops, const int64_t* lds,
                            const float* ta, hs_cand* out, const int64_t* out_offsets,
                            const int64_t* caps, int64_t* counts, void* stream)
{
    if (!p || p->n_fops < 1 || !fops || !lds || !ta || !out || !out_offsets || !caps || !counts)
        return HS_ERR_INVALID;
    try {
        hipStream_t s = (hipStream_t)stream;
        DevTabs t;
        const hs_status st = device_tables(p, s, &t);
        if (st != HS_OK) return st;
        if (hsk::launch_zero_i64(counts, (int64_t)p->n_fops * (p->H + 1), s) != hipSuccess) return HS_ERR_HIP;
        hsk::WalkArgs a = walk_args(p, t.walk);
        a.n_fops = p->n_fops;
        a.fops = fops;
        a.lds = lds;
        a.out_offsets = out_offsets;
        a.caps = caps;
        a.ta = ta;
        a.out = out;
        a.counts = reinterpret_cast<unsigned long long*>(counts);
        return from_hip(launch_detect(p, a, s));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

size_t hs_sort_workspace_bytes(int64_t n)
{
    if (n <= 1) return 0;
    size_t bytes = 0;
    if (hsk::sort_workspace(n, &bytes) != hipSuccess) return 0;
    return bytes;
}

hs_status hs_sort_candidates(hs_cand* cand, int64_t n, void* work, void* stream)
{
    if (n < 0 || (n > 1 && (!cand || !work))) return HS_ERR_INVALID;
    try {
        return from_hip(hsk::sort_candidates(reinterpret_cast<uint64_t*>(cand), n, work,
                                             (hipStream_t)stream));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

namespace {
size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }
size_t plane_bytes(const hs_plan* p) { return (size_t)p->T * (size_t)p->N * 4; }
size_t partial_bytes(const hs_plan* p)
{
    return (size_t)hsk::backward_partial_floats((int)p->T, p->H, p->N, true) * 4;
}
bool tau_ok(float tau) { return tau > 0.0f && tau < INFINITY; }
}  // namespace

size_t hs_backward_workspace_bytes(const hs_plan* p)
{
    if (!p || p->n_fops != 0) return 0;
    return round256(partial_bytes(p));
}

hs_status hs_sum_backward(const hs_plan* p, const float* g, float* dfop, void* work, void* stream)
{
    if (!p || p->n_fops != 0 || !g || !dfop) return HS_ERR_INVALID;
    if (p->mapping != HS_MAP_PAPER) return HS_ERR_UNSUPPORTED;
    if (partial_bytes(p) > 0 && !work) return HS_ERR_INVALID;
    try {
        return from_hip(hsk::launch_backward(g, dfop, static_cast<float*>(work), (int)p->T, p->N, p->H,
                                             (hipStream_t)stream));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

// Workspace of the statistic: the backward's partial rows and the fused
// forward's per-block pairs;
// for 16-bit plans also the H planes the forward materialises, followed by
// the larger of the partials and the plane reduction's pairs.
size_t hs_lse_workspace_bytes(const hs_plan* p)
{
    if (!p || p->n_fops != 0) return 0;
    const size_t bwd = (size_t)hsk::backward_partial_floats((int)p->T, p->H, p->N, false) * 4;
    const size_t fused = (size_t)hsk::kLseMaxBlocks * p->H * 2 * sizeof(float);
    if (p->dtype == HS_DTYPE_F32) return std::max(round256(bwd), round256(fused));
    const size_t tail = std::max(bwd, (size_t)hsk::lse_part_bytes(p->H));
    return round256(plane_bytes(p) * p->H) + round256(tail);
}

namespace {

// Grid of the fused statistic: two blocks per compute unit (the planner's
// LDS budget), at most one per tile and kLseMaxBlocks.
int lse_grid(const hs_plan* p)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    int64_t g = p->persistent_blocks > 0 ? p->persistent_blocks : 2 * (int64_t)cus;
    g = std::min<int64_t>(g, std::min<int64_t>(p->tiles_total, hsk::kLseMaxBlocks));
    return (int)std::max<int64_t>(g, 1);
}

// The fused statistic (fp32 plans): the planes are formed tile by tile and
// never stored; `part` holds lse_grid(p) x H (max, sum) pairs.
hs_status lse_forward_fused(const hs_plan* p, const void* fop, int64_t ld, float tau, double* lse, double* loss,
                            float* part, const DevTabs& t, hipStream_t s)
{
    const int g = lse_grid(p);
    hsk::TileArgs a = tile_args(p, fop, ld, t);
    a.lse_part = part;
    a.lse_c = (float)(1.4426950408889634 / (double)p->scale / (double)tau);
    hipError_t e = hsk::launch_fused(hsk::kModeLse, p->dtype, p->H, a, p->tiles_total, g, p->lds_bytes, s);
    if (e != hipSuccess) return HS_ERR_HIP;
    e = hsk::launch_lse_fused_final(a.lse_part, g, p->H, 1.0 / (double)p->scale, (double)tau, lse, s);
    if (e != hipSuccess) return HS_ERR_HIP;
    return loss ? from_hip(hsk::launch_lse_loss(lse, p->H, (double)tau, loss, s)) : HS_OK;
}

}  // namespace

hs_status hs_lse_forward_noalloc(const hs_plan* p, const void* fop, int64_t ld, float tau, double* lse,
                                 double* loss, void* stream)
{
    if (!p || p->n_fops != 0 || !lse || !tau_ok(tau)) return HS_ERR_INVALID;
    if (p->mapping != HS_MAP_PAPER || p->dtype != HS_DTYPE_F32) return HS_ERR_UNSUPPORTED;
    if (!fop_ok(p, fop, ld, p->N)) return HS_ERR_INVALID;
    try {
        hipStream_t s = (hipStream_t)stream;
        if ((size_t)lse_grid(p) * p->H * 2 * sizeof(float) > hsk::kNoAllocScratchBytes) return HS_ERR_INVALID;
        void* scratch = nullptr;
        if (hsk::noalloc_scratch(&scratch) != hipSuccess) return HS_ERR_HIP;
        DevTabs t;
        const hs_status st = device_tables_present(p, s, &t);
        if (st != HS_OK) return st;
        return lse_forward_fused(p, fop, ld, tau, lse, loss, static_cast<float*>(scratch), t, s);
    } catch (...) {
        return HS_ERR_HIP;
    }
}

hs_status hs_lse_forward(const hs_plan* p, const void* fop, int64_t ld, float tau, double* lse,
                         double* loss, void* work, void* stream)
{
    if (!p || p->n_fops != 0 || !lse || !work || !tau_ok(tau)) return HS_ERR_INVALID;
    if (p->mapping != HS_MAP_PAPER) return HS_ERR_UNSUPPORTED;
    if (!fop_ok(p, fop, ld, p->N)) return HS_ERR_INVALID;
    try {
        hipStream_t s = (hipStream_t)stream;
        DevTabs t;
        const hs_status st = device_tables(p, s, &t);
        if (st != HS_OK) return st;
        if (p->dtype == HS_DTYPE_F32) return lse_forward_fused(p, fop, ld, tau, lse, loss, static_cast<float*>(work), t, s);
        float* planes = static_cast<float*>(work);
        void* tail = static_cast<char*>(work) + round256(plane_bytes(p) * p->H);
        hsk::TileArgs a = tile_args(p, fop, ld, t);
        a.hp = planes;
        hipError_t e = hsk::launch_fused(hsk::kModeSum, p->dtype, p->H, a, p->tiles_total,
                                         p->persistent_blocks, p->lds_bytes, s);
        if (e != hipSuccess) return HS_ERR_HIP;
        e = hsk::launch_lse_reduce(planes, p->T * p->N, p->H, tau, tail, lse, s);
        if (e != hipSuccess) return HS_ERR_HIP;
        return loss ? from_hip(hsk::launch_lse_loss(lse, p->H, (double)tau, loss, s)) : HS_OK;
    } catch (...) {
        return HS_ERR_HIP;
    }
}

hs_status hs_lse_backward(const hs_plan* p, const void* fop, int64_t ld, const double* lse,
                          float tau, const double* gscale, float* dfop, void* work, void* stream)
{
    if (!p || p->n_fops != 0 || !lse || !dfop || !work || !tau_ok(tau)) return HS_ERR_INVALID;
    if (p->mapping != HS_MAP_PAPER) return HS_ERR_UNSUPPORTED;
    if (!fop_ok(p, fop, ld, p->N)) return HS_ERR_INVALID;
    try {
        // the weights are formed inside the transpose's first pass: no weight
        // plane is written or read back
        return from_hip(hsk::launch_lse_backward_fused(p->dtype, fop, ld, (int)p->T, p->N, p->H, 1.0f / p->scale,
                                                       (double)tau, lse, gscale, dfop, static_cast<float*>(work),
                                                       (hipStream_t)stream));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

hs_status hs_check_counts(const int64_t* counts_host, int32_t n_hp, int64_t capacity)
{
    if (!counts_host || n_hp < 1 || n_hp > hsk::kMaxH || capacity < 0) return HS_ERR_INVALID;
    if (counts_host[n_hp] < 0) return HS_ERR_INVALID;
    return counts_host[n_hp] > capacity ? HS_ERR_OVERFLOW : HS_OK;
}

const char* hs_status_string(hs_status s)
{
    switch (s) {
    case HS_OK: return "ok";
    case HS_ERR_INVALID: return "invalid argument";
    case HS_ERR_OVERFLOW: return "candidate list exceeds capacity";
    case HS_ERR_HIP: return "HIP runtime error";
    case HS_ERR_UNSUPPORTED: return "unsupported";
    case HS_ERR_NOMEM: return "out of memory";
    }
    return "unknown status";
}

hs_status hs_stream_read(const void* src, int64_t bytes, float* sink, int32_t grid, void* stream)
{
    if (!src || !sink || bytes <= 0 || bytes % 16 != 0 || (reinterpret_cast<uintptr_t>(src) & 15) != 0 ||
        grid < 1 || grid > 65536)
        return HS_ERR_INVALID;
    try {
        return from_hip(hsk::launch_stream_read(src, bytes, sink, grid, (hipStream_t)stream));
    } catch (...) {
        return HS_ERR_HIP;
    }
}

const char* hs_version(void) { return "hs-mi355x 0.1.0 (gfx950)"; }

}  // extern "C"
