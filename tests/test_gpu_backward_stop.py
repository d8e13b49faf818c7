"""The adjoint ends a ray at the sample where the forward ended it, also where
t_stop is the forward's own T or the float next to it, so that one last place in
a sample's exp(-sigma delta) would show.  Without a network, and with all voxels
of the samples stored, the colour gradients of a ray add up to
g (1 - T) with T that of its last sample: one sample too few or too many moves
the sum by at least 0.2 (1 - exp(-0.05 * 50 / 192)) = 2.6e-3, float sums of at
most 100 terms by 1e-5.  Bar: 1e-3.  sigma_scale / N and sigma_scale * (1 / N)
differ for these N."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2103_14645_amd import snerg as S
from tests.gpu_helpers import handle, say

pytestmark = pytest.mark.gpu


def grid(N, B):
    G = N // B
    dens = np.random.default_rng(N).uniform(0.05, 0.3, (N, N, N)).astype(np.float32)
    dens[:2] = dens[-2:] = dens[:, :2] = dens[:, -2:] = dens[:, :, :2] = dens[:, :, -2:] = 0.0
    blocks = dens.reshape(G, B, G, B, G, B).transpose(0, 2, 4, 1, 3, 5).reshape(G ** 3, B, B, B)
    n = G ** 3
    return S.DeviceGrid(handle(), N, B, np.arange(n, dtype=np.int32), np.ascontiguousarray(blocks),
                        np.full((n, B, B, B, 3), 0.5, np.float32), np.zeros((n, B, B, B, 4), np.float32),
                        sigma_scale=50.0), n * B ** 3


@pytest.mark.parametrize("N,B", [(96, 32), (192, 32)])
@pytest.mark.parametrize("mode", ["scattered", "patch", "dense view", "sparse view"])
def test_adjoint_stops_with_the_forward(mode, N, B):
    say(f"stop of the adjoint: {mode}, N={N}")
    assert np.float32(50) / np.float32(N) != np.float32(50) * (np.float32(1) / np.float32(N))
    dg, nv = grid(N, B)
    h, mlp = handle(), S.mlp_tensor(W.mlp_weights())
    out, aux = torch.empty((1, 4), device="cuda"), torch.empty((1, 8), device="cuda")
    g = torch.tensor([[1.0, 0.0, 0.0, 0.0]], device="cuda")
    gm, gg = torch.empty(883, device="cuda"), torch.empty((nv, 8), device="cuda")
    ids = torch.zeros(1, dtype=torch.int64, device="cuda") if mode in ("scattered", "patch") else None
    fov = 120.0 if mode == "sparse view" else 0.01
    for seed in range(16):
        carr = S.make_cameras([W.orbit_camera(1, 1, fov, seed=seed)])

        def opts(t):
            return S.make_opts(mlp_on=False, t_stop=t, bg=(0.0, 0.0, 0.0), patch_rays=mode == "patch", grad_packed=True)

        def forward(t):
            S.snerg_render(h, dg.struct(), mlp, carr, ids, 1, opts(t), out, aux)
            return float(aux[0, 7])

        last = np.float32(forward(0.3))
        assert 0.2 < last < 0.3
        for t in (float(last), float(np.nextafter(last, np.float32(1)))):
            T = forward(t)
            S.snerg_render_backward(h, dg.struct(), mlp, carr, ids, 1, opts(t), aux, g, gm, gg, None, None)
            got = float(gg[:, 1].double().sum())
            assert abs(got - (1.0 - T)) < 1e-3, (mode, N, seed, t, T, got)
