// C entries to the launch rules of csrc/routes.h, for tests/test_routes.py.
#include "routes.h"

using namespace snerg;

extern "C" {

int route_dense_view(const double* eye, double focal, int N) { return dense_view(eye, focal, N); }

int route_backward(int keys, int listed, int ids, int patch, int dense, int64_t lds, int64_t rays) {
    return int(backward_route(keys != 0, listed != 0, ids != 0, patch != 0, dense != 0, lds, rays));
}

int route_render(int N, int B, int list, int64_t rays, int64_t pixels, int f32, int f16) {
    const RenderSplit s = render_split(N, B, list != 0, rays, pixels, f32 != 0, f16 != 0);
    return 2 * s.lanes + s.ordered;
}

}  // extern "C"
