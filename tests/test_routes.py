"""The rules by which calls are dealt to kernels (csrc/routes.h), compiled for
the host and checked over the forms that they accept."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2103_14645_amd", "csrc")
LOGS, LISTED, EIGHT, ONE = range(4)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("routes") / "libroutes.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC,
                    os.path.join(HERE, "host_routes.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def dense(lib, eye, focal, N):
    e = np.ascontiguousarray(eye, dtype=np.float64)
    return bool(lib.route_dense_view(e.ctypes.data_as(ctypes.c_void_p), ctypes.c_double(focal), N))


def test_dense_views(lib):
    # outside the grid: a pixel covers |eye| / focal at the centre, a voxel 2 / N
    for d, focal, want in ((2.0, 512.0, True), (2.0, 511.0, False), (4.0, 1024.0, True), (4.0, 1000.0, False)):
        assert dense(lib, (0.0, d, 0.0), focal, 512) == want, (d, focal)
    # inside it, at the faces: an eye in the middle does not make wide pixels dense
    for eye in ((0.0, 0.0, 0.0), (0.05, -0.02, 0.1), (0.5, 0.5, 0.5)):
        assert not dense(lib, eye, 80.0, 512)
        assert dense(lib, eye, 256.0, 512)


def adjoint_lds(G):
    return -(-G ** 3 // 32) * 8 + 512 * 9 * 4 + 512


@pytest.mark.parametrize("G", [1, 16, 63, 64])
@pytest.mark.parametrize("rays", [64, 38400, 65536, 1 << 40])
def test_backward_routes(lib, G, rays):
    i64 = ctypes.c_int64
    for keys, listed, ids, patch, dense_ in itertools.product((0, 1), repeat=5):
        if listed and not (ids and keys):
            continue
        got = lib.route_backward(keys, listed, ids, patch, dense_, i64(adjoint_lds(G)), i64(rays))
        if not keys:
            want = LOGS
        elif listed:
            want = LISTED
        elif ids and not patch:  # long scattered lists keep the order of one lane per ray
            want = ONE
        elif G == 64 and rays > 38400:  # a workgroup of 32 rays would have the compute unit to itself
            want = ONE
        else:
            want = EIGHT if dense_ else ONE
        assert got == want, (keys, listed, ids, patch, dense_)


def split(lib, N, B, rays, list_=False, f32=False, f16=False, pixels=5120000):
    i64 = ctypes.c_int64
    return lib.route_render(N, B, int(list_), i64(rays), i64(pixels), int(f32), int(f16)) // 2


SHAPES = [(N, B) for B in (2, 4, 8, 16, 32, 64) for N in range(B, min(64 * B, 2048) + 1, B) if N // B in (1, 2, 8, 16, 32, 40, 48, 56, 64)]


@pytest.mark.parametrize("f32,f16", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_render_launches_hold_fewer_than_2_to_32_lanes(lib, f32, f16):
    for N, B in SHAPES:
        for list_ in (0, 1):
            for e in range(6, 34):
                for rays in ((1 << e) - 64, 1 << e, (1 << e) + 64):
                    lanes = split(lib, N, B, rays, list_, f32, f16)
                    assert lanes in ((1, 2, 4, 16) if f32 else (1, 4, 16))
                    assert lanes == 1 or rays * lanes < 1 << 32, (N, B, list_, rays, lanes)


# Where several lanes to a ray were measured to lose against one (and where they win).
@pytest.mark.parametrize("N,B,rays,kw,lanes", [
    (128, 2, 16384, {}, 1), (128, 2, 4096, {}, 16), (64, 2, 65536, {}, 1), (64, 2, 16384, {}, 16),
    (256, 4, 65536, {}, 1), (256, 4, 16384, dict(f16=True), 1), (256, 4, 4096, {}, 16), (64, 4, 65536, {}, 4),
    (512, 8, 65536, {}, 1), (512, 8, 163840, {}, 1), (512, 8, 16384, {}, 16), (256, 8, 65536, {}, 4),
    (1024, 16, 65536, dict(list_=True), 1), (512, 16, 65536, dict(list_=True), 4),
    (512, 32, 4096, {}, 16), (512, 32, 65536, dict(list_=True), 4), (512, 32, 262144, {}, 4), (512, 32, 640000, {}, 1),
    (256, 4, 65536, dict(f32=True, f16=True), 1), (256, 4, 640000, dict(f32=True), 1),
    (512, 8, 163840, dict(f32=True), 1), (512, 8, 5120000, dict(f32=True), 1),
    (64, 8, 640000, dict(f32=True, f16=True), 1), (64, 8, 5120000, dict(f32=True), 1),
    (256, 16, 2560000, dict(f32=True, f16=True), 1), (512, 32, 5120000, dict(f32=True), 2),
    (512, 16, 152551, dict(list_=True), 1), (512, 16, 152551, dict(list_=True, pixels=664000), 4),
    (256, 16, 110000, dict(f16=True), 4), (192, 32, 162000, dict(f16=True), 4), (48, 8, 89088, dict(f16=True), 4),
    (1024, 32, 65536, dict(f32=True, f16=True, list_=True), 4), (512, 32, 1 << 20, dict(f32=True, list_=True), 4),
])
def test_render_lanes(lib, N, B, rays, kw, lanes):
    assert split(lib, N, B, rays, **kw) == lanes
