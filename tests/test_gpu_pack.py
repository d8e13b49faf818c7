"""The packed grid byte for byte: occupancy words, rank maps, padded voxels
and distance bytes, against NumPy (exact: every value is an integer or a
copy)."""
import numpy as np
import pytest
import torch
from scipy import ndimage

from paper_2103_14645_amd import snerg as S
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def align256(x):
    return (x + 255) & ~255


def expected(N, B, ind, dens, rgb, feat):
    """(bits, ranks) of the occupancy words, rank_lin, rank_id, distance bytes
    [r, z, y, x] and padded voxels [r, z, y, x, 8]."""
    G, n = N // B, len(dens)
    lin = np.nonzero((ind >= 0) & (ind < n))[0]
    occ = np.zeros(-(-G ** 3 // 32) * 32, np.uint8)
    occ[lin] = 1
    bits = np.packbits(occ.reshape(-1, 32), axis=1, bitorder="little").view(np.uint32).reshape(-1)
    ranks = np.concatenate([[0], np.cumsum(occ.reshape(-1, 32).sum(1))[:-1]]).astype(np.int32)
    rank_lin = np.full(n, -1, np.int32)
    rank_id = np.full(n, -1, np.int32)
    lin = lin[:n]
    rank_lin[:len(lin)] = lin
    rank_id[:len(lin)] = ind[lin]
    full = np.zeros((N + 2,) * 3 + (8,), dens.dtype)
    for b in np.nonzero((ind >= 0) & (ind < n))[0]:
        z, y, x = (1 + B * int(c) for c in (b // (G * G), b // G % G, b % G))
        full[z:z + B, y:y + B, x:x + B] = np.concatenate(
            [dens[ind[b]][..., None], rgb[ind[b]], feat[ind[b]]], -1)
    vox = np.zeros((n, B + 2, B + 2, B + 2, 8), dens.dtype)
    dist = np.full((n, B + 1, B + 1, B + 1), 255, np.uint8)
    for r, b in enumerate(lin):
        z, y, x = (B * int(c) for c in (b // (G * G), b // G % G, b % G))
        vox[r] = full[z:z + B + 2, y:y + B + 2, x:x + B + 2]
        d = vox[r, ..., 0] != 0
        act = np.zeros((B + 1,) * 3, bool)
        for c in range(8):
            act |= d[c >> 2:B + 1 + (c >> 2), (c >> 1) & 1:B + 1 + ((c >> 1) & 1), c & 1:B + 1 + (c & 1)]
        if act.any():
            dist[r] = ndimage.distance_transform_cdt(~act, metric="chessboard")
    return bits, ranks, rank_lin, rank_id, dist, vox


def check(N, B, ind, dens, rgb, feat):
    dg = S.DeviceGrid(H.handle(), N, B, ind, dens, rgb, feat)
    torch.cuda.synchronize()
    raw = dg.packed.cpu().numpy()
    n, G = len(dens), N // B
    words = -(-G ** 3 // 32)
    bits, ranks, rank_lin, rank_id, dist, vox = expected(N, B, ind, dens, rgb, feat)
    occ = raw[:8 * words].view(np.uint32).reshape(-1, 2)
    assert np.array_equal(occ[:, 0], bits)
    assert np.array_equal(occ[:, 1].view(np.int32), ranks)
    off = align256(8 * words)
    assert np.array_equal(raw[off:off + 4 * n].view(np.int32), rank_lin)
    off += align256(4 * n)
    assert np.array_equal(raw[off:off + 4 * n].view(np.int32), rank_id)
    off += align256(4 * n)
    cells, item = (B + 1) ** 3, dens.dtype.itemsize
    dist_bytes = (cells + 15) & ~15
    size = (B + 2) ** 3 * 8 * item
    stride = align256(dist_bytes + size)
    for r in range(n):
        rec = raw[off + r * stride:off + (r + 1) * stride]
        assert np.array_equal(rec[:cells].reshape(dist[r].shape), dist[r]), (N, B, r)
        got = rec[dist_bytes:dist_bytes + size].view(dens.dtype).reshape(vox[r].shape)
        assert np.array_equal(got, vox[r]), (N, B, r)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("N,B", [(2, 2), (14, 2), (20, 4), (24, 8), (64, 8), (48, 16), (32, 32), (96, 32), (128, 64)])
def test_packed_bytes(N, B, f32):
    H.say(f"pack N={N} B={B} f32={f32}")
    rng = np.random.default_rng(N * 100 + B)
    G = N // B
    n = max(1, min(G ** 3, 20))
    ind = np.full(G ** 3, -1, np.int32)
    ind[rng.choice(G ** 3, n, replace=False)] = rng.permutation(n)
    dens = np.where(rng.random((n, B, B, B)) < 0.3, rng.integers(1, 256, (n, B, B, B)), 0)
    # blocks that are empty, hold one voxel at a corner, or a lone plane: the longest distances
    dens[0] = 0
    if n > 2:
        dens[1] = 0
        dens[1, 0, 0, 0] = 7
        dens[2] = 0
        dens[2, B - 1] = 9
    t = np.float32 if f32 else np.uint8
    rgb, feat = rng.integers(0, 256, (n, B, B, B, 3)), rng.integers(0, 256, (n, B, B, B, 4))
    check(N, B, ind, dens.astype(t), rgb.astype(t), feat.astype(t))


@pytest.mark.parametrize("f32", [False, True])
def test_packed_bytes_odd_indirection(f32):
    """Atlas ids out of range, unused and repeated; more macroblocks than one pass of the table."""
    B, G = 2, 40
    N, n = B * G, 300
    rng = np.random.default_rng(5)
    ind = np.where(rng.random(G ** 3) < 0.004, rng.integers(0, n, G ** 3), -1).astype(np.int32)
    ind[::997] = n + 3
    t = np.float32 if f32 else np.uint8
    dens, rgb, feat = (rng.integers(0, 3, (n, B, B, B) + c).astype(t) for c in ((), (3,), (4,)))
    check(N, B, ind, dens, rgb, feat)
    # every macroblock names one of few ids: ranks beyond n_blocks are dropped
    check(N, B, (np.arange(G ** 3) % n).astype(np.int32), dens, rgb, feat)


@pytest.mark.parametrize("G", [23, 24, 25, 33, 63, 64])
def test_tables_of_small_and_large_grids(G):
    # the occupancy words and rank maps by one workgroup and by the whole chip
    N, B = 2 * G, 2
    rng = np.random.default_rng(G)
    lin = rng.permutation(G ** 3)[:40]
    ind = np.full(G ** 3, -1, np.int32)
    ind[lin] = rng.permutation(43)[:40]  # three atlas entries that no macroblock holds
    dens, rgb, feat = (rng.integers(0, 256, (43, B, B, B) + s, dtype=np.uint8) for s in ((), (3,), (4,)))
    check(N, B, ind, dens, rgb, feat)


def test_more_records_than_one_launch_holds():
    """110,592 uint8 records of blocks of 32 (39 GB): their padded voxels are more than
    2^32 threads.  The colour and density arrays are parts of the feature array, so
    that the canonical values take 14.5 GB."""
    N, B = 1536, 32
    G = N // B
    n = G ** 3
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB of device memory")
    H.say(f"pack of {n} records")
    feat = torch.empty(4 * n * B ** 3, dtype=torch.uint8, device="cuda")
    ramp = (torch.arange(1 << 20, device="cuda") * 131 >> 3).to(torch.uint8)
    feat.view(-1, 1 << 20).copy_(ramp)
    feat.view(n, -1).add_(torch.arange(n, device="cuda").to(torch.uint8)[:, None])
    ids = torch.from_numpy(np.random.default_rng(0).permutation(n).astype(np.int32)).cuda()
    packed = torch.empty(S.snerg_packed_size(N, B, n, S.SNERG_U8), dtype=torch.uint8, device="cuda")
    S.snerg_pack_grid(H.handle(), N, B, n, S.SNERG_U8, ids, feat, feat, feat, packed)
    torch.cuda.synchronize()
    off = align256(8 * (n // 32)) + 2 * align256(4 * n)
    dist_bytes, size = (33 ** 3 + 15) & ~15, 34 ** 3 * 8
    stride = align256(dist_bytes + size)
    for r in (0, 1, 54321, 108941, 108942, n - 1):
        at = off + r * stride + dist_bytes
        vox = packed[at:at + size].view(34, 34, 34, 8)[1:33, 1:33, 1:33]
        i, B3 = int(ids[r]), B ** 3
        for lo, hi, per in ((0, 1, 1), (1, 4, 3), (4, 8, 4)):
            want = feat[per * i * B3:per * (i + 1) * B3].view(B, B, B, per)
            assert torch.equal(vox[..., lo:hi], want), (r, lo)
    del feat, packed, vox, want
    torch.cuda.empty_cache()
