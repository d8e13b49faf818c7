// Which kernel a call takes: the rules that look at sizes alone, free of the
// device so that they can be checked without one.
#pragma once

#include <cmath>
#include <cstdint>

namespace snerg {

// How a render deals rays to lanes: lanes per ray, and whether its tiles go in
// heavy-first order.
struct RenderSplit {
    int32_t lanes, ordered;
};

// Lanes per ray, by measurement (us; views of a shell grid at 39 degrees,
// scattered pixels, 8x8 patches).  uint8, 512^3:
//                       1 lane    4     16
//    4,096 pixels/patches  402/180  175/83  74/47
//   32,768                 339/235  181/105 169/110
//   65,536                 382/296  222/140 272/178
//   512x512 frame          394     266 (in tile order; 352 in image order)
//   640x480 frame          372     323        (1024^3: 859 -> 576)
//   1250x200, all on it    257     218        1250x300: 274 -> 306
//   800x800 frame          412     530        (1024^3, FP16: 859 -> 1084)
// so 16 lanes up to 2^15 rays, 4 up to 5 2^16.  One lane's time is that of the
// longest ray, in proportion to N, four lanes' more and more the chip's, in
// proportion to the rays, so on smaller grids the line lies lower, and with
// small macroblocks, whose walk every lane of a ray repeats (one lane, four):
// 512^3 in blocks of 16, 1250x250 325, 404; 320^3, 187,500 rays 180, 158,
// 375,000 238, 278; 128^3, 120,000 rays 163, 105, 187,500 126, 141; 64^3,
// 86,000 51, 35, 110,600 55, 57; 96^3 in blocks of 4, 81,000 99, 114.  Past 2^16
// rays the wavefronts are not all resident at once, and the order pays for its
// two launches, but not up to 192^3 (120,000 rays 131 in order, 124 without).
// float32 samples are 256 bytes each and bound by the texture
// path; the samples of one ray side by side share most of their lines, so
// there the split also pays where the chip is full: eight 800x800 views of
// the 512^3 grid 5.25 ms, 2 lanes 4.05, 4 lanes 5.1; of a 1024^3 grid 13.0,
// 7.6, 7.9; 2^20 scattered pixels 3.38, 2.09, 1.95.  The FP16 network's tiles
// run once per wavefront, however many rays it holds: four 1080p views take
// 7.05 ms with one lane and 7.20 with two, eight 800x800 views 5.24 and 4.86.
//
// rays: of a list its entries, of views 64 for each tile, since a wavefront is
// launched and its tables are staged however few of them lie in the image.
inline RenderSplit render_split(int32_t N, int32_t B, bool list, int64_t rays, bool f32, bool f16) {
    if (rays <= (int64_t(1) << 15)) return {16, 0};
    if (rays <= (int64_t(1) << 16)) return {4, 0};
    const int64_t most = N < 128   ? (B < 8 ? int64_t(1) << 16 : int64_t(3) << 15)
                         : N < 192 ? int64_t(1) << 17
                         : N < 512 || B < 32 ? int64_t(3) << 16
                                             : int64_t(5) << 16;
    if (rays <= most) return {4, N > 192};
    if (f32 && list && rays <= (int64_t(1) << 20)) return {4, 1};
    // (a launch holds fewer than 2^32 lanes)
    if (f32 && rays <= (f16 ? int64_t(6) << 20 : int64_t(1) << 30)) return {2, 1};
    return {1, 1};
}

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
