// Strip-walk detection kernel for gfx950: harmonic planes (Eq. 1-2 of
// arXiv:1805.12258, Sec. III) thresholded into packed candidates, with no
// plane written to memory.
//
// Work decomposition.  The plane is cut into strips of B = 64 V consecutive
// bins (V = 2, 4 or 8 bins per lane, a template parameter chosen per plan).
// A wave walks runs of rows of a strip (hs_rows.h); waves are independent.
//
// Order.  A host-built schedule lists the strips of each XCD (blocks are
// dealt to the XCDs in turn): the strips are dealt to eight lists by the
// three bits after the leading one of the strip index, and each list is
// ordered by position inside the octave, so that strips x, x/2, x/4 and x/8
// are summed on one XCD at nearly the same time; lists of uneven length are
// then evened out.  A batch assigns whole FOPs to XCDs first.
#pragma once

#include "hs_rows.h"

namespace hsk {
namespace walk {

// Largest threshold table of a plan that the strip walk takes; taller planes
// run as the tile kernel's strips of four bins per lane.  The walk itself has no
// such limit: the line says which plans report the strip walk, and by which
// pitch a batch rejects a FOP.
constexpr int kWThrBytes = 16384;

__host__ __device__ constexpr int thr_stride(int H) { return (H + 3) & ~3; }

}  // namespace walk

template <typename TIn, int H, int V>
__global__ __launch_bounds__((64 * rows::block_waves(H, rows::lane_bins(H, V))),
                             (rows::min_waves(H, rows::lane_bins(H, V)))) void k_walk(WalkArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    rows::walk_plan<TIn, H, V, false>(a, smem);
}

// The same over a batch (a kernel of its own: the walk has no scalar registers
// to spare for a batch's place in its list where there is none).
template <typename TIn, int H, int V>
__global__ __launch_bounds__((64 * rows::block_waves(H, rows::lane_bins(H, V))),
                             (rows::min_waves(H, rows::lane_bins(H, V)))) void k_walk_batch(WalkArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    rows::walk_plan<TIn, H, V, true>(a, smem);
}

template <typename TIn, int H, int V>
hipError_t launch_walk_t(const WalkArgs& a, int grid, hipStream_t s)
{
    return rows::launch_plan(a.n_fops > 0 ? k_walk_batch<TIn, H, V> : k_walk<TIn, H, V>, H, V, a, grid, s);
}

}  // namespace hsk
