"""The gradient of a grid of 2^31 voxels and more, whose indices the summing tables
cannot hold: whole views, patches, scattered rays and rays with more samples than
are listed go through the wavefronts' logs with 64-bit indices, with atlas ids on
both sides of voxel 2^31.  8,300 blocks of 64^3, of which eight hold anything and
are read: 79 GB packed and 70 GB of gradients, the values parts of one array of
35 GB that is never filled.  Bar as in test_gpu_backward_paths.py."""
import gc

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from paper_2103_14645_amd import snerg as S
from tests.gpu_helpers import handle, say
from tests.test_gpu_backward import compare

pytestmark = pytest.mark.gpu

N, B, N_BLOCKS = 1344, 64, 8300
G, B3 = N // B, B ** 3
IDS = [0, 8299, 5, 8192, 8191, 77, 4000, 8298]  # 8192 B^3 = 2^31


@pytest.fixture(scope="module")
def grid():
    gc.collect()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GB of device memory")
    rng = np.random.default_rng(31)
    ind = np.full(G ** 3, -1, np.int32)
    for i, atlas in enumerate(IDS):
        ind[((10 + (i >> 2)) * G + 10 + ((i >> 1) & 1)) * G + 10 + (i & 1)] = atlas
    flat = torch.empty(4 * N_BLOCKS * B3, device="cuda")
    for atlas in IDS:
        for per in (1, 3, 4):
            v = rng.random(per * B3, dtype=np.float32)
            if per == 1:
                v = np.where(rng.random(B3) < 0.3, v, np.float32(0))
            flat[per * atlas * B3:per * (atlas + 1) * B3] = torch.from_numpy(v).cuda()
    part = [[flat[per * a * B3:per * (a + 1) * B3].cpu().numpy() for a in IDS] for per in (1, 3, 4)]
    vals = tuple(np.stack(p).reshape((len(IDS), B, B, B) + s) for p, s in zip(part, ((), (3,), (4,))))
    small = np.full(G ** 3, -1, np.int32)
    for i, atlas in enumerate(IDS):
        small[ind == atlas] = i
    d_ind = torch.from_numpy(ind).cuda()
    packed = torch.empty(S.snerg_packed_size(N, B, N_BLOCKS, S.SNERG_F32), dtype=torch.uint8, device="cuda")
    S.snerg_pack_grid(handle(), N, B, N_BLOCKS, S.SNERG_F32, d_ind, flat, flat, flat, packed)
    torch.cuda.synchronize()
    st = S.snerg_grid(N, B, N_BLOCKS, S.SNERG_F32, d_ind.data_ptr(), packed.data_ptr(), 50.0, 0)
    grad = torch.zeros((N_BLOCKS * B3, 8), device="cuda")
    yield st, O.OracleGrid(W.Grid(N, B, small, None, None, None), values=vals), grad
    del flat, packed, grad, d_ind
    gc.collect()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("mlp_on", [True, False])
@pytest.mark.parametrize("mode", ["views", "sparse views", "scattered", "patch", "long rays"])
def test_logs_with_64_bit_indices(grid, mode, mlp_on):
    st, og, grad = grid
    say(f"backward of a grid of 2^31 voxels: {mode}, mlp={mlp_on}")
    if mode == "long rays":  # along the diagonal, three of four samples active
        cams = [W.look_at((1.2, 1.2, 1.2), 5, 4, 1.0)]
    else:
        cams = [W.orbit_camera(37, 29, 9.0, seed=3), W.orbit_camera(9, 20, 9.0, seed=4)]
    if mode == "sparse views":
        cams = [W.orbit_camera(160, 120, 120.0, seed=5)]
    total = sum(c.n_rays for c in cams)
    ids = None
    if mode in ("scattered", "patch", "long rays"):
        ids = np.random.default_rng(1).permutation(total)[:total - 3]
    n = total if ids is None else len(ids)
    mlp = W.mlp_weights(5)
    g_rgba = (np.random.default_rng(2).normal(size=(n, 4)) / n).astype(np.float32)
    opts = S.make_opts(early_stop=False, mlp_on=mlp_on, patch_rays=mode == "patch", grad_packed=True, accumulate=True)
    carr, m = S.make_cameras(cams), S.mlp_tensor(mlp)
    d_ids = torch.from_numpy(ids).cuda() if ids is not None else None
    out, aux = torch.empty((n, 4), device="cuda"), torch.empty((n, 8), device="cuda")
    gm = torch.zeros(883, device="cuda")
    S.snerg_render(handle(), st, m, carr, d_ids, n, opts, out, aux)
    assert float((aux[:, 7] >= 0).float().mean()) > (0.001 if mode == "sparse views" else 0.05)
    S.snerg_render_backward(handle(), st, m, carr, d_ids, n, opts, aux, torch.from_numpy(g_rgba).cuda(), gm, grad, None,
                            None)
    got = np.stack([grad[a * B3:(a + 1) * B3].cpu().numpy() for a in IDS]).reshape(len(IDS), B, B, B, 8)
    for a in IDS:  # the next test starts from zero again
        grad[a * B3:(a + 1) * B3] = 0
    om, od, orr, of = O.render_grad(og, mlp, cams, g_rgba, ray_ids=ids, early_stop=False, mlp_on=mlp_on)
    compare("mlp", gm.cpu().numpy(), om)
    compare("dens", got[..., 0], od)
    compare("rgb", got[..., 1:4], orr)
    compare("feat", got[..., 4:8], of)
