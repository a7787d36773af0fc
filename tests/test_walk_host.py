"""CPU test of the dense walk (csrc/rmpc_dense.h, built for the host) against the oracle, ray by ray: hits,
float64 distances and visits equal, flags equal but for near-ties, which the walk may leave out.
The box entries are the test's own, by distance transforms of the bricks' occupancy."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest
from scipy import ndimage

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which(HIPCC) is None:
        pytest.skip("hipcc not available")
    so = str(tmp_path_factory.mktemp("walk") / "libwalk.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2301_08068_amd", "csrc"),
                    os.path.join(HERE, "walk_host.hip"), "-o", so], check=True, capture_output=True)
    return C.CDLL(so)


def _reach(occ, walls, flat=None):
    """Half extent (at most 15) of the free square (perpendicular to axis `flat`) or cube around every
    brick: the chessboard distance to an occupied one, past a walled end of an axis (those of `walls`)
    everything is occupied."""
    s = np.ones((3, 3, 3), bool)
    if flat is not None:
        for end in (0, 2):
            s[tuple(end if a == flat else slice(None) for a in range(3))] = False
    pad = np.pad(occ, [(0, int(w)) for w in walls], constant_values=True)
    d = ndimage.distance_transform_cdt(~pad, s) if pad.any() else np.full(pad.shape, 15)
    d = np.where(d < 0, 15, d)                                     # (a plane without an occupied brick)
    return np.minimum(d, 15)[tuple(slice(0, n) for n in occ.shape)]


def _entries(occ, whole):
    """Box entries [nbz, nby, nbx] of an occupancy [nz, ny, nx]; whole: of whole bricks only."""
    nb = [n // 2 if whole else -(-n // 2) for n in occ.shape]
    walls = [2 * b < n for b, n in zip(nb, occ.shape)]
    pad = np.zeros([2 * b for b in nb], bool)
    part = occ[:2 * nb[0], :2 * nb[1], :2 * nb[2]]
    pad[:part.shape[0], :part.shape[1], :part.shape[2]] = part
    vox = pad.reshape(nb[0], 2, nb[1], 2, nb[2], 2)
    mask = sum(vox[:, (b >> 2) & 1, :, (b >> 1) & 1, :, b & 1].astype(np.int64) << b for b in range(8))
    e = _reach(mask > 0, walls).astype(np.int64)
    best, code = np.zeros(nb, np.int64), np.full(nb, 1 << 8 | 3 << 9)
    for a in range(3):                                             # x, y, z; array axis 2 - a
        for side in range(2):
            layer = np.take(vox, side, axis=2 * (2 - a) + 1)
            r = _reach(layer.any(axis=tuple(i for i, n in enumerate(layer.shape) if i in _subs(2 - a))), walls, 2 - a)
            code = np.where(r > best, side << 8 | a << 9, code)
            best = np.maximum(best, r)
    return np.where(mask > 0, 0x8000 | mask | code | best << 11, 2 * e * (1 | 1 << 5 | 1 << 10)).astype(np.uint16)


def _subs(dropped):
    """Positions of the sub-voxel axes left in a [b, 2, b, 2, b, 2] array without that of axis `dropped`."""
    left = [(i, k) for i in range(3) for k in range(2) if (i, k) != (dropped, 1)]
    return [p for p, (_, k) in enumerate(left) if k == 1]


def _check(lib, occ, g, rmax, dirs, h=1.0, segments=(1, 2, 4, 8, 16)):
    t = np.where(occ, -0.1, 0.3).astype(np.float32)
    g = np.asarray(g, np.float32)
    dirs = np.ascontiguousarray(dirs, np.float32)
    n = len(dirs)
    o = oracle.trace(oracle.OracleMap(t, h, np.zeros(3), "f32"), g, dirs, rmax, nthreads=4)
    dims = np.array(occ.shape[::-1], np.int32)
    for whole in (False, True) if any(k % 2 for k in occ.shape) else (False,):
        e = np.ascontiguousarray(_entries(occ, whole))
        bricks = np.array(e.shape[::-1], np.int32)
        for S in segments:
            if S > 1 and rmax / h / S < 4:
                continue
            hit, visits = np.zeros(n, np.int32), np.zeros(n, np.int32)
            d, flags = np.zeros(n), np.zeros(n, np.uint8)
            p = [a.ctypes.data_as(C.c_void_p) for a in (t, e, dims, bricks, g)]
            out = [a.ctypes.data_as(C.c_void_p) for a in (hit, d, flags, visits)]
            assert lib.walk_rays(*p, C.c_double(h), C.c_double(rmax), dirs.ctypes.data_as(C.c_void_p), n, S, *out), "a walk does not end"
            label = f"{occ.shape} whole {whole} S {S} g {g} range {rmax}"
            assert np.array_equal(hit, o["hit"]), label
            assert np.array_equal(d[hit >= 0], o["d"][hit >= 0]) and np.all(np.isinf(d[hit < 0])), label
            assert np.array_equal(visits, o["visits"]), label
            assert np.array_equal(flags & 6, o["flags"] & 6) and not np.any(flags & 1 & ~o["flags"]), label


def _free(rng, occ, whole=False):
    """A start in a free voxel: anywhere, on a face or in a centre."""
    k = np.argwhere(~occ)
    at = k[rng.integers(len(k))][::-1].astype(np.float64)
    return at + (rng.integers(0, 2, 3) * 0.5 if whole else rng.uniform(0.0, 1.0, 3).astype(np.float32))


@pytest.mark.parametrize("density", [0.0, 0.002, 0.02, 0.15, 0.5])
def test_random_grids(lib, density):
    """Grids of odd and even extents, free ones to half full, ranges that end anywhere or on faces."""
    rng = np.random.default_rng(int(1000 * density))
    dirs = oracle.directions(600)
    for k in range(24):
        occ = rng.uniform(size=rng.integers(1, 50, 3)) < density
        if occ.all():
            continue
        if k % 3 == 0:
            occ[:, occ.shape[1] // 2] |= rng.uniform(size=occ[:, 0].shape) < 0.9      # a plate to graze
            if occ.all():
                continue
        rmax = float(rng.integers(1, 40)) if k % 2 else float(rng.uniform(1.0, 60.0))
        _check(lib, occ, _free(rng, occ, k % 4 == 0), rmax, dirs)


def test_structured_directions(lib):
    """Axis-aligned, diagonal and vanishing directions, from faces and centres, where crossings tie."""
    d = np.array([[i, j, k] for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1) if i or j or k], np.float32)
    unit = d / np.linalg.norm(d, axis=1, keepdims=True)
    dirs = np.concatenate([unit, unit * np.float32([1, 1e-20, 1]), unit * np.float32([1e-38, 1, 1e-41])]).astype(np.float32)
    dirs = dirs[np.linalg.norm(dirs, axis=1) > 0.5]
    rng = np.random.default_rng(2)
    for k in range(30):
        occ = rng.uniform(size=(31, 40, 33)) < 0.03
        _check(lib, occ, _free(rng, occ, k % 3 > 0), float(rng.integers(3, 50)), dirs)


@pytest.mark.parametrize("shape", [(3, 6, 4000), (4000, 5, 4), (7, 3999, 2)])
def test_long_lines(lib, shape):
    """Lines of 4,000 voxels, where a float32 crossing is off by a thousandth of a voxel: rays along
    them, a little off the axis and off its diagonal, and all round."""
    rng = np.random.default_rng(sum(shape))
    along = 2 - int(np.argmax(shape))
    occ = rng.uniform(size=shape) < 0.0005
    dirs = rng.normal(size=(400, 3)) * 0.0015
    dirs[:, along] = rng.choice([-1.0, 1.0], 400)
    dirs = np.concatenate([dirs / np.linalg.norm(dirs, axis=1, keepdims=True), oracle.directions(200)])
    for k in range(6):
        _check(lib, occ, _free(rng, occ, k % 3 == 0), [5000.0, 777.0, 2600.5][k % 3], dirs)


@pytest.mark.parametrize("off", [0.0, 2e-6, 8e-6, 9.9e-6, 1.1e-5, 1.9e-5, 3e-5])
@pytest.mark.parametrize("shape,faces", [((9, 12, 10), 1), ((9, 12, 10), 5), ((33, 70, 35), 2), ((33, 70, 35), 30)])
def test_range_near_ties(lib, shape, faces, off):
    """Ranges that end just before and behind faces that rays along and across the axes reach, in grids
    where the walk knows a float32 position better than to 1e-5 voxel and where it does not: the
    decision, and the flag of a crossing within 1e-5 voxel of the range."""
    rng = np.random.default_rng(faces)
    d = np.array([[i, j, k] for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1) if i or j or k], np.float64)
    dirs = np.concatenate([d / np.linalg.norm(d, axis=1, keepdims=True),
                           rng.uniform(-1.0, 1.0, (200, 3)) * [0.2, 1.0, 0.2]])
    dirs[26:] /= np.linalg.norm(dirs[26:], axis=1, keepdims=True)
    slant = np.abs(dirs[26:].astype(np.float32)[:, 1]).astype(np.float64)
    for density in (0.0, 0.02):
        occ = rng.uniform(size=shape) < density
        mid = [n // 2 for n in shape]
        occ[tuple(slice(k - 1, k + 2) for k in mid)] = False
        g = np.array([mid[2], mid[1] + 0.5, mid[0] + 0.5])
        for sign in (-1.0, 1.0):
            for reach in [float(faces), faces - 0.5] + list((faces - 0.5) / slant[:3]):
                _check(lib, occ, g, reach + sign * off, dirs, segments=(1, 4))
