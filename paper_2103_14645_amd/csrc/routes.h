// Which kernel a call takes: the rules that look at sizes alone, free of the
// device so that they can be checked without one.
#pragma once

#include <cmath>
#include <cstdint>

namespace snerg {

// Whether a camera's pixels lie no further apart than the voxels where the
// grid is: at its centre, or for an eye inside the grid at its faces, which the
// rays still have ahead of them (a 160x160 view of 90 degrees from the middle of
// a 512^3 grid has 3 voxels to a pixel there).
inline bool dense_view(const double eye[3], double focal, int32_t N) {
    const double d = std::sqrt(eye[0] * eye[0] + eye[1] * eye[1] + eye[2] * eye[2]);
    return (d > 1.0 ? d : 1.0) * N <= 2.0 * focal;
}

// How a backward call takes its rays.
enum class BackwardRoute : int32_t {
    kLogs,           // eight lanes to a ray, through the wavefronts' logs
    kListed,         // a list of samples first: patches or scattered rays
    kEightLanes,     // eight lanes to a ray, a workgroup's table
    kOneLane,        // one lane to a ray, a wavefront's table
};

// keys: the grid's voxels fit the tables' keys.  listed: a ray list short enough
// that the launch keeps its samples.  ids: a ray list; patch: in groups of 64
// neighbours.  dense: every camera a dense_view.  lds: bytes a workgroup of the
// eight-lane kernel takes (occupancy table and summing table); rays: those of the
// list, or 64 for each tile.
//
// Eight lanes halve the time (eight 800x800 views, 512^3: 17.5 against 27 ms; two
// of 160x160: 2.2 against 4.5 for the whole call; 270,000 rays in patches 3.9
// against 1.4), but they enter the table in another order.  Where a tile's voxels
// don't fit the table, order decides what overflows and goes unrounded, and the
// feature gradients would differ by the table's own rounding: 4e-5 of their norm
// for 160x160 views of a 512^3 grid, 2.2e-5 for 270,000 scattered rays of it, but
// 1.5e-6 for 800x800 views and 1.7e-6 for 270,000 rays in patches.  So views whose
// pixels are further apart than the voxels and long scattered lists take one lane.
//
// At 64^3 macroblocks the occupancy table alone is 64 KB, and a workgroup of 32
// rays has the compute unit to itself, where one lane to a ray has 256 on it: four
// 800x800 views of 128^3 in blocks of 2 take 32.4 ms with eight lanes and 16.9 with
// one, of 512^3 in blocks of 8 50.6 and 34.6 (at 63^3, where two workgroups fit,
// 16.7 and 16.7, 26.1 and 34.5).  As long as the launch is a few workgroups per
// compute unit eight lanes still win: two 160x120 views 1.0 and 1.1 ms, 2.5 and 3.9;
// one of 256x256 1.16 and 1.07, of 1024^3 in blocks of 16 7.3 and 5.8.
constexpr int64_t kCuLds = 160 << 10;

inline BackwardRoute backward_route(bool keys, bool listed, bool ids, bool patch, bool dense, int64_t lds,
                                    int64_t rays) {
    if (!keys) return BackwardRoute::kLogs;
    if (listed) return BackwardRoute::kListed;
    if (!dense || (ids && !patch)) return BackwardRoute::kOneLane;
    if (2 * lds > kCuLds && rays > (5 << 13)) return BackwardRoute::kOneLane;
    return BackwardRoute::kEightLanes;
}

}  // namespace snerg
