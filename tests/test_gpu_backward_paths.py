"""The gradient of the grid through each of the kernels that a backward call
can take, at the sizes where their rules change: views whose pixels are closer
than the voxels and views whose pixels are further apart, with odd image sizes;
ray lists in patches and scattered, of 1 to a few more than whole groups of
rays, over so many voxels that a group's table fills and is emptied on the way.
Bar: |g_gpu - g_oracle| <= 1e-4 * max|g_oracle| + 1e-7 per element: float32
values through up to 2^7 samples a ray, fixed-point sums to 2^-24 of the
largest gradient a hand-over."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_helpers import say
from tests.test_gpu_backward import compare, run_backward, shadow_values

pytestmark = pytest.mark.gpu


def check(cams, mlp_on, ids=None, patch=False):
    g = W.tiny_grid(n_occupied=200, seed=21)
    vals = shadow_values(g, 21)
    mlp = W.mlp_weights(22)
    n = sum(c.n_rays for c in cams) if ids is None else len(ids)
    g_rgba = np.random.default_rng(23).normal(size=(n, 4)) / n
    kw = dict(early_stop=False, mlp_on=mlp_on)
    gm, gd, gr, gf, _ = run_backward(g, vals, mlp, cams, g_rgba, ids=ids, patch_rays=patch, **kw)
    om, od, orr, of = O.render_grad(O.OracleGrid(g, values=vals), mlp, cams, g_rgba, ray_ids=ids, **kw)
    compare("mlp", gm, om)
    compare("dens", gd, od)
    compare("rgb", gr, orr)
    compare("feat", gf, of)


@pytest.mark.parametrize("mlp_on", [True, False])
@pytest.mark.parametrize("width,height,fov", [(65, 33, 20.0), (65, 33, 90.0), (8, 8, 60.0), (1, 9, 5.0)])
def test_views_of_close_and_of_sparse_pixels(width, height, fov, mlp_on):
    cams = [W.orbit_camera(width, height, fov, seed=3), W.orbit_camera(height, width, fov, seed=4)]
    say(f"views {width}x{height}, {fov} degrees, focal {cams[0].focal:.0f}, mlp={mlp_on}")
    check(cams, mlp_on)


@pytest.mark.parametrize("mlp_on", [True, False])
@pytest.mark.parametrize("patch", [True, False])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1037])
def test_lists_of_whole_and_ragged_groups(n, patch, mlp_on):
    cams = [W.orbit_camera(48, 40, 70.0, seed=5)]
    ids = np.random.default_rng(n).permutation(cams[0].n_rays)[:n]
    check(cams, mlp_on, ids=ids, patch=patch)
