"""The autotuner where a ray has several lanes: only the tile of a launch shape
counts there, so the other fields stay what they were."""
import pytest
import torch

import workloads as W
from paper_2103_14645_amd import snerg as S
from tests.gpu_helpers import device_grid, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("persistent", [False, True])
def test_small_renders_leave_the_unmeasured_fields(persistent):
    say(f"autotune of a thumbnail, persistent={persistent}")
    dg = device_grid(W.tiny_grid(n_occupied=64, seed=1))
    h = S.Handle()
    opts, m = S.make_opts(persistent=persistent), S.mlp_tensor(W.mlp_weights())
    small = S.make_cameras([W.orbit_camera(64, 48, seed=2)])
    large = S.make_cameras([W.orbit_camera(700, 640, seed=2)])
    out = torch.empty((700 * 640, 4), device="cuda")
    for own in ((8, 8, 1, 2), (8, 8, 2, 16)):
        S.snerg_set_tuning(h, *own)
        best, _ = S.snerg_autotune(h, dg.struct(), m, small, opts, out, reps=1)
        assert best[2:] == own[2:]
        now = S.snerg_tuning_lookup(h, dg.struct(), large, opts)
        assert now == (best, False)  # what a render of another size falls back to
    best, _ = S.snerg_autotune(h, dg.struct(), m, small, opts, out, candidates=[(16, 4, 4, 8), (16, 4, 1, 3)], reps=1)
    assert best == (16, 4, 4, 8)
    assert S.snerg_tuning_lookup(h, dg.struct(), large, opts) == ((16, 4, 2, 16), False)
    # one lane to a ray: the whole shape is measured and kept
    best, _ = S.snerg_autotune(h, dg.struct(), m, large, opts, out, candidates=[(16, 4, 4, 8), (16, 4, 1, 3)], reps=1)
    assert best in ((16, 4, 4, 8), (16, 4, 1, 3))
    other = S.make_cameras([W.orbit_camera(699, 640, seed=2)])
    assert S.snerg_tuning_lookup(h, dg.struct(), other, opts) == (best, False)
