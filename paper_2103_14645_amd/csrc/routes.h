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

// Lanes per ray.  A render of few rays is a few wavefronts per SIMD, each as long
// as its longest ray (in proportion to N), and several lanes to a ray make it
// shorter; of many rays it is bound by the chip's throughput, which they lower:
// every lane of a ray repeats its walk over the macroblocks (in proportion to
// N / B), a workgroup of 256 lanes stages the whole occupancy table (8 KB at 32^3
// macroblocks, 64 KB at 64^3, where two workgroups fill a compute unit) for 16 or
// 64 rays, and the FP16 network's tiles run once per wavefront, however many rays
// it holds.  One lane's time over that of 16 / of 4, uint8, slowest to fastest of
// shells and random blocks, both networks (a list: scattered over 40 to 160 times as
// many pixels; one lane goes 16 or 32 rays to a wavefront there):
//   rays            16,384             32,768             65,536             131,072
//   N, B       view 16   view 4   view 16   list 4    view 4    list 4    view 4
//   64, 2      1.06-1.4  0.7-1.0  0.65-0.85 0.7-0.9   0.7-1.1   0.65-0.7
//   128, 2     0.44-0.9  0.45-1.0 0.24-0.5  0.8-1.0   0.3-0.65
//   64, 4      1.5-1.7   1.3-1.5  0.9-1.05  0.9-1.2   1.0-1.3   0.8-1.0   0.8-0.9
//   256, 4     0.74-1.4  0.9-1.1  0.4-0.8   0.8-1.1   0.3-0.7
//   128, 8     2.0-2.1   1.5-1.7  1.3-1.4   0.9-1.4   1.2-1.4   0.8-1.0   0.9-1.05
//   256, 8     2.3-3.1   1.05-1.7 1.5-2.0   1.1-1.25  1.1-1.5   0.96-1.1  0.8-1.1
//   512, 8     1.0-2.1   1.3-1.4  0.5-1.3   1.05-1.2  0.4-0.8
//   256, 16    2.7-4.0   1.6-2.5  1.8-2.5   1.3-1.8   1.5-2.1   1.2-1.4   1.1-1.4
//   768, 16    2.4-4.2   1.5-1.8  1.4-2.9   1.3-1.4   0.8-1.9             0.6-1.5
//   1024, 16   1.4-2.8   1.5-1.6  0.8-1.9   1.4-1.5   0.5-1.1
//   256, 32    3.1-4.2   2.6-2.8  2.1-2.6   1.8-2.1   1.7-2.4   1.6-1.7   1.3-1.6
//   512, 32    4.0-5.5   2.2-2.6  2.9-3.7   1.75-1.9  2.1-2.4   1.5-1.7   1.4-2.0
//   1024, 32   4.7-5.6   2.0-2.3  3.1-4.1   1.7-1.9   2.0-2.4   1.45-1.6  1.4-2.3
// Lists of 131,072 scattered rays 0.78-0.9 in blocks of 16, 0.94-1.4 in blocks of 32;
// where they take more than a sixteenth of the pixels, or come in patches, rays share
// samples as a view's do (512, 16, 152,551 of 664,000 pixels: 523 us, 364).  Views of
// 313,600 0.9-1.1 for 512, 32 and 1.1-1.5 for 1024, 32.  Past 2^16 rays the wavefronts
// are not all resident at once, and the tile order pays for its two launches, but not
// up to 192^3 (128^3, 120,000 rays 131 us in order, 124 without).
// float32 samples are 256 bytes each and bound by the texture path; the samples of
// one ray side by side share most of their lines, so there the split also pays
// where the chip is full, unless macroblocks are small.  One lane over 2 lanes,
// eight 800x800 views, FP32 / FP16 network: 64, 32 0.95 / 0.88; 128, 32 1.11 / 0.99;
// 512, 32 1.24 / 1.02; 1024, 32 1.71 / 1.52; 512, 16 0.98 / 0.81; 256, 8 0.87 / 0.72;
// 560x560: 128, 16 1.22 / 1.13; 512, 16 1.35 / 1.23; 128, 8 1.06 / 0.98.  Over 4:
// 560x560 192, 32 1.38 / 1.22; 512, 32 2.0 / 1.7; 512, 16 1.45 / 1.25; 512, 8 0.55 /
// 0.4; 2^20 scattered rays 128, 32 1.3 / 1.1; 64, 32 1.05 / 0.96; 512, 16 1.2 / 0.96.

// For blocks under 8 and tables of more than 8 KB (G = N / B over 32).  Each network
// counts here, so work is in rays with the FP32 one.
inline RenderSplit render_split_small_blocks(int32_t N, int32_t B, bool list, int64_t rays, bool f32, bool f16) {
    constexpr int64_t K = 1 << 10, M = 1 << 20;
    const int32_t G = N / B;
    const int table = G <= 40 ? 0 : (G <= 56 ? 1 : 2);  // the occupancy table: up to 16, 43, 64 KB
    const int64_t work = f16 ? rays + rays / 4 : rays;
    auto at_most = [](int64_t& line, int64_t v) { line = line < v ? line : v; };

    int64_t most16 = B < 8 ? 16 * K : (B < 16 ? 32 * K : 48 * K);
    if (table > 0) at_most(most16, B < 4 || (B < 8 && table > 1) ? 8 * K : (B < 8 ? 16 * K : 24 * K));
    if ((list ? 2 * work : work) <= most16) return {16, 0};

    int64_t most4 = 0, most2 = 0;
    if (!f32) {
        if (B == 4) most4 = N <= 64 ? 64 * K : 0;
        else if (B >= 8) most4 = table == 0 ? 64 * K : (table > 1 ? 24 * K : (B > 8 ? 48 * K : 32 * K));
        if (list) most4 /= 2;
    } else if (list) {
        if (B >= 4) most4 = B < 16 ? 64 * K : (B == 16 ? 512 * K : 1280 * K);
        if (table == 1) at_most(most4, B < 8 ? 32 * K : (B < 16 ? 64 * K : (f16 ? 80 * K : 512 * K)));
        if (table == 2) at_most(most4, B < 8 ? 16 * K : (B < 16 ? 32 * K : 40 * K));
        if (B >= 16) most2 = B > 16 ? (f16 ? 5 * M : 1 << 30) : (table == 0 ? M : 0);
    } else {
        if (B >= 4) most4 = B < 8 ? 64 * K : (B < 16 ? 96 * K : (B == 16 ? 384 * K : M));
        if (table == 1 && B < 16) at_most(most4, 64 * K);
        if (table == 2) at_most(most4, B < 8 ? 24 * K : (B < 16 ? 40 * K : (f16 ? 48 * K : 160 * K)));
        if (B == 16) most2 = table == 0 ? 768 * K : (table == 1 || !f16 ? 384 * K : 0);
        else if (B > 16) most2 = f16 ? 7 * M : 1 << 30;
    }
    if (work <= most4) return {4, work > 64 * K && N > 192};
    if (work <= most2) return {2, 1};
    return {1, 1};
}

// rays: of a list its entries, of views 64 for each tile, since a wavefront is
// launched and its tables are staged however few of them lie in the image.
// pixels: of all cameras.
inline RenderSplit render_split(int32_t N, int32_t B, bool list, int64_t rays, int64_t pixels, bool f32, bool f16) {
    constexpr int64_t K = 1 << 10, M = 1 << 20;
    if (B < 8 || N / B > 32) return render_split_small_blocks(N, B, list, rays, f32, f16);

    const int64_t most16 = list ? (B == 8 ? 24 * K : 32 * K) : (N < 512 || B == 8 ? 34 * K : (B == 16 ? 48 * K : 64 * K));
    if (rays <= most16) return {16, 0};

    const bool sparse = list && rays * 16 < pixels;
    int64_t most4, most2 = 0;
    if (!f32) {
        if (N < 128) most4 = sparse && B == 8 ? 64 * K : 96 * K;
        else if (B == 8) most4 = sparse ? 40 * K : 80 * K;
        else if (N < 192) most4 = sparse ? (B == 16 ? 80 * K : 110 * K) : 128 * K;
        else if (B == 16) most4 = sparse ? 80 * K : (f16 ? 200 * K : 208 * K);
        else most4 = N < 512 ? 208 * K : 336 * K;
    } else if (list) {
        if (B == 8) most4 = f16 ? 52 * K : 64 * K;
        else most4 = B == 16 || N < 128 ? (f16 ? 400 * K : 512 * K) : M;
        if (B == 16) most2 = f16 ? 0 : M;
        else if (B > 16) most2 = f16 ? 6 * M : 1 << 30;
    } else {
        if (B == 8) most4 = N < 128 ? 96 * K : (f16 ? 130 * K : 160 * K);
        else if (N < (B == 16 ? 256 : 128)) most4 = 160 * K;
        else most4 = B == 16 || N < 512 ? 384 * K : (N < 1024 && B == 32 ? 512 * K : M);
        if (B == 8) most2 = N / B > 16 ? 0 : (N < 128 ? 160 * K : (f16 ? 320 * K : 384 * K));
        else if (N < 128 || (B == 16 && f16)) most2 = 512 * K;
        else most2 = f16 ? (N < 512 ? 2 * M : 6 * M) : 1 << 30;
    }
    if (rays <= most4) return {4, rays > 64 * K && N > 192};
    // (a launch holds fewer than 2^32 lanes)
    if (rays <= most2) return {2, 1};
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
// Eight lanes take less time (whole calls, 512^3, one lane against eight: eight
// 800x800 views 23.4 and 16.4 ms, two of 160x160 3.0 and 0.9, 270,000 rays in patches
// 3.1 and 1.2, scattered 4.2 and 2.9), but they enter the table in another order.  Where a tile's voxels
// don't fit the table, order decides what overflows and goes unrounded, and the
// feature gradients would differ by the table's own rounding: 4e-5 of their norm
// for 160x160 views of a 512^3 grid, 2.2e-5 for 270,000 scattered rays of it, but
// 1.5e-6 for 800x800 views and 1.7e-6 for 270,000 rays in patches.  So views whose
// pixels are further apart than the voxels and long scattered lists take one lane.
//
// At 64^3 macroblocks the occupancy table alone is 64 KB, and a workgroup of 32
// rays has the compute unit to itself, where one lane to a ray has 256 on it: eight
// 800x800 views of 128^3 in blocks of 2 take 65 ms with eight lanes and 32 with one,
// of 512^3 in blocks of 8 96 and 60 (at 63^3, where two workgroups fit, 33.6 and 32,
// 49 and 59).  As long as the launch is a few workgroups per compute unit eight
// lanes still win: two 160x120 views 0.94 and 0.97 ms, 2.1 and 3.25; one of 256x256
// of the 128^3 grid 1.11 and 0.94.
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
