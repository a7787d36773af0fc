"""The C-ABI library builds, loads and exports every entry point the header declares
(no GPU calls: these run on the CPU)."""
import ctypes as C
import os
import re
import subprocess

import numpy as np

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "rmpcast.h")


def _declared():
    text = open(HEADER).read()
    return sorted(set(re.findall(r"^\s*(?:rmpc_status|const char \*)\s*(rmpc_\w+)\s*\(", text, re.M)))


@pytest.fixture(scope="module")
def lib_path():
    from paper_2301_08068_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    return build.LIB


def test_header_declares_the_boundary():
    names = _declared()
    for must in ("rmpc_create", "rmpc_destroy", "rmpc_map_upload", "rmpc_map_release", "rmpc_query",
                 "rmpc_scan_query", "rmpc_trace_debug", "rmpc_directions", "rmpc_last_error"):
        assert must in names


def test_library_exports_every_declared_symbol(lib_path):
    out = subprocess.run(["nm", "-D", "--defined-only", lib_path], capture_output=True, text=True,
                         check=True).stdout
    exported = set(re.findall(r"\sT\s(rmpc_\w+)$", out, re.M))
    missing = [n for n in _declared() if n not in exported]
    assert not missing, missing


def test_library_resolves_its_own_symbols(lib_path):
    """No entry point or kernel launcher is left undefined (a shared library links even when
    one of its sources was not compiled in)."""
    out = subprocess.run(["nm", "-D", "--undefined-only", lib_path], capture_output=True, text=True,
                         check=True).stdout
    assert not re.findall(r"rmpc", out), out


def test_binding_loads_and_resolves(lib_path):
    from paper_2301_08068_amd import binding
    assert set(binding.exported_symbols()) == set(_declared())
    assert binding._lib.rmpc_last_error() == b""


def test_library_has_no_oracle_dependency(lib_path):
    """The product library neither links nor names the oracle."""
    out = subprocess.run(["nm", "-D", lib_path], capture_output=True, text=True, check=True).stdout
    assert "orc_" not in out
    ldd = subprocess.run(["ldd", lib_path], capture_output=True, text=True).stdout
    assert "rmp_oracle" not in ldd
    for f in os.listdir(os.path.join(ROOT, "paper_2301_08068_amd")):
        if f.endswith(".py"):
            src = open(os.path.join(ROOT, "paper_2301_08068_amd", f)).read()
            assert "import oracle" not in src and "from oracle" not in src, f


def test_map_footprint_and_size_limits(lib_path):
    """rmpc_map_footprint makes no GPU call: the dense layout is the grid, then one summary
    element per whole 8^3 cell and per whole 2^3 brick, each section starting on a multiple of
    256 elements; grids of 2^31 voxels or more are refused (int32 linear indices)."""
    from paper_2301_08068_amd import binding
    fp = binding.rmpc_map_footprint
    n = 400 ** 3
    cell_base = -(-n // 256) * 256
    brick_base = -(-(cell_base + 50 ** 3) // 256) * 256
    assert fp(400, 400, 400, "f32", 0.05, (0, 0, 0)) == 4 * (brick_base + 200 ** 3)
    assert fp(400, 400, 400, "u8", 0.05, (0, 0, 0)) == brick_base + 200 ** 3
    # ragged grid: partial cells and bricks have no summary
    assert fp(13, 7, 9, "f16", 0.1, (0, 0, 0)) == 2 * (1024 + 6 * 3 * 4)     # 819 voxels, no whole cell
    assert fp(1290, 1290, 1290, "u8", 0.01, (0, 0, 0)) > 0             # 2.147e9 - 1.2e6 voxels
    with pytest.raises(binding.RmpcError, match="2\\^31"):
        fp(1291, 1291, 1291, "u8", 0.01, (0, 0, 0))                     # 2.1518e9 voxels
    with pytest.raises(binding.RmpcError, match="dimensions"):
        fp(4097, 1, 1, "u8", 0.01, (0, 0, 0))
    with pytest.raises(binding.RmpcError, match="voxel size"):
        fp(8, 8, 8, "f32", float("nan"), (0, 0, 0))


def test_sparse_workload_round_trip():
    """The sparse-map inputs the GPU tests compare against the oracle: blocks cut from a dense
    map and expanded again give back the dense occupancy (free blocks dropped or kept), at any
    block offset, and stored values keep their block layout (block, z, y, x)."""
    from paper_2301_08068_amd import workloads as W
    m = W.tiny_map(1)
    for off, keep in (((0, 0, 0), 0.0), ((-5, 3, -2), 0.5)):
        sm = W.sparse_from_dense(m, offset_blocks=off, keep_free=keep, seed=4)
        lo = np.asarray(off) * 8
        dense, origin = sm.dense_crop(lo, lo + 64)
        assert np.array_equal(dense <= 0, m.tsdf <= 0)
        assert np.allclose(origin, m.origin_m)
        assert np.all(np.any(sm.values <= 0, axis=(1, 2, 3)) | (keep > 0))
    k = int(np.argmax(np.any(sm.values <= 0, axis=(1, 2, 3))))
    bx, by, bz = sm.coords[k] - np.asarray((-5, 3, -2))
    assert np.array_equal(sm.values[k], m.tsdf[8 * bz:8 * bz + 8, 8 * by:8 * by + 8, 8 * bx:8 * bx + 8])


@pytest.mark.parametrize("n", [0, 1, 3, 4, 63, 64, 65, 130])
def test_result_columns_equal_single_results(lib_path, n):
    """The conversion of an array of results equals that of each result alone, byte for byte."""
    from paper_2301_08068_amd import binding as B
    rng = np.random.default_rng(n)
    out = (B.Result * max(n, 1)).from_buffer_copy(rng.bytes(B.RESULT_BYTES * max(n, 1)))
    rows = B.result_dicts(out, n)
    assert len(rows) == n
    for r, d in zip(out, rows):
        one = B.result_dict(r)
        assert list(d) == list(one)
        for k in one:
            assert type(d[k]) is type(one[k]) and np.shape(d[k]) == np.shape(one[k])
            assert np.asarray(d[k]).tobytes() == np.asarray(one[k]).tobytes()
        for k, field in (("f", r.f), ("S", r.A), ("b", r.b), ("lam", r.lam)):
            assert d[k].tobytes() == bytes(field) and d[k].flags.writeable
        assert (d["rank"], d["flags"], d["visits"]) == (r.rank, r.flags, r.visits)


class _MapView(C.Structure):
    _fields_ = [("data", C.c_void_p), ("box", C.c_void_p)] + \
        [(k, C.c_int32) for k in ("nx", "ny", "nz", "dtype", "nbx", "nby", "nbz", "partial", "lo", "span")]


@pytest.mark.parametrize("dims", [(400, 400, 400), (64, 64, 64), (130, 130, 130), (8, 4096, 4096), (1, 4096, 4096),
                                  (2, 2048, 2048), (16, 2000, 2000), (6, 7, 4096), (4096, 1, 4096), (8, 8, 8), (1, 1, 1)])
def test_upload_scratch_is_bounded(lib_path, dims):
    """The scratch of an upload: a byte and 52 bits a brick of 2^3 voxels, rows of bits padded to 64
    bricks along the axis where that costs least: below 14 bytes a brick, and 2 MiB."""
    scratch = C.CDLL(lib_path)._ZN4rmpc17box_scratch_bytesERKNS_7MapViewE
    scratch.restype = C.c_size_t
    nb = [-(-n // 2) for n in dims]
    m = _MapView(nx=dims[0], ny=dims[1], nz=dims[2], nbx=nb[0], nby=nb[1], nbz=nb[2])
    assert scratch(C.byref(m)) < 14 * nb[0] * nb[1] * nb[2] + (2 << 20)


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 3, 4), (5, 7, 9), (16, 6, 1)])
def test_host_entries_of_single_bricks(lib_path, dims):
    """The entries that the host makes of uint8 voxels when there is no scratch: the voxels of an
    occupied brick, a box of one brick around a free one."""
    fill = C.CDLL(lib_path)._ZN9rmpc_host15host_unit_boxesERKN4rmpc7MapViewEPKhPt
    fill.restype = None
    nx, ny, nz = dims
    nb = [-(-n // 2) for n in dims]
    vox = (np.random.default_rng(sum(dims)).uniform(size=(nz, ny, nx)) < 0.2).astype(np.uint8) * 7
    out = np.full((nb[2], nb[1], nb[0]), 0xabcd, np.uint16)
    m = _MapView(nx=nx, ny=ny, nz=nz, nbx=nb[0], nby=nb[1], nbz=nb[2])
    fill(C.byref(m), vox.ctypes.data_as(C.c_void_p), out.ctypes.data_as(C.c_void_p))
    mask = np.zeros(out.shape, np.int64)
    for z, y, x in np.argwhere(vox):
        mask[z // 2, y // 2, x // 2] |= 1 << (x % 2 + 2 * (y % 2) + 4 * (z % 2))
    assert np.array_equal(out, np.where(mask > 0, mask | 0x8700, 2 * (1 | 1 << 5 | 1 << 10)))
