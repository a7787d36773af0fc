"""The box entries of an uploaded map (csrc/box_kernels.hip): one 16-bit entry per brick of 2 x 2 x 2
voxels, read back from the arena and checked against the grid brick by brick."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ARENA = 96 << 20
OCCUPIED, SIDE, AXIS, EXTENT = 0x8000, 8, 9, 11


def _fill(B, ctx, dev, keep):
    """Leave room in the arena for one map of `keep` bytes and less than 4 KiB more."""
    held = B.rmpc_map_upload(ctx, 4096, 1, -(-keep // 4096), "u8", 0.1, (0, 0, 0), dev, True)
    n = 4096
    while n:
        try:
            B.rmpc_map_upload(ctx, 256, n, 16, "u8", 0.1, (0, 0, 0), dev, True)
        except B.RmpcError as e:
            assert e.status == B.RMPC_E_NOMEM
            n //= 2
    n = 16
    while n:
        try:
            B.rmpc_map_upload(ctx, 256, 1, n, "u8", 0.1, (0, 0, 0), dev, True)
        except B.RmpcError as e:
            assert e.status == B.RMPC_E_NOMEM
            n //= 2
    B.rmpc_map_release(ctx, held)


def _entries(B, torch, grid, dtype, source="device"):
    """Entries [nbz, nby, nbx] of a grid [nz, ny, nx] uploaded into a fresh arena, from device memory
    ("device"; "offset": one element past an aligned address; "tight": into an arena that has no room
    but for the map) or from "host" memory."""
    arena = torch.zeros(ARENA, dtype=torch.uint8, device="cuda:0")
    ctx = B.rmpc_create(0, arena.data_ptr(), ARENA)
    nz, ny, nx = grid.shape
    try:
        raw = torch.from_numpy(grid.view(np.uint8).reshape(-1))
        shift = grid.dtype.itemsize if source == "offset" else 0
        dev = torch.cat([torch.zeros(shift, dtype=torch.uint8), raw]).to("cuda:0")
        if source == "tight":
            full = B.rmpc_map_footprint(nx, ny, nz, dtype, 0.1, (0.0, 0.0, 0.0))
            zeros = torch.zeros(256 * 4096 * 16, dtype=torch.uint8, device="cuda:0")
            _fill(B, ctx, zeros.data_ptr(), -(-full // 256) * 256)
        before = arena.clone()
        ptr = raw.data_ptr() if source == "host" else dev.data_ptr() + shift
        B.rmpc_map_upload(ctx, nx, ny, nz, dtype, 0.1, (0.0, 0.0, 0.0), ptr, source != "host")
        raw = arena.cpu().numpy()
        base = int(torch.nonzero(arena != before)[0]) // 256 * 256
    finally:
        B.rmpc_destroy(ctx)
    n, eb = nx * ny * nz, grid.dtype.itemsize
    whole = (nx // 2) * (ny // 2) * (nz // 2)
    cell_base = -(-n // 256) * 256
    room = (-(-(cell_base + (nx // 8) * (ny // 8) * (nz // 8)) // 256) * 256 + whole - cell_base) * eb
    nb = [-(-k // 2) for k in (nx, ny, nz)]
    off = base
    if dtype != "u8":
        assert np.array_equal(raw[base:base + n * eb], grid.view(np.uint8).reshape(-1)), "the grid is kept as given"
        off = base + cell_base * eb
        if 2 * nb[0] * nb[1] * nb[2] > room:
            nb = [nx // 2, ny // 2, nz // 2]
    k = nb[0] * nb[1] * nb[2]
    return raw[off:off + 2 * k].view(np.uint16).reshape(nb[2], nb[1], nb[0])


def _sum(a):
    """Prefix sums with a leading zero along each axis."""
    s = np.zeros(tuple(n + 1 for n in a.shape), np.int64)
    s[1:, 1:, 1:] = a.cumsum(0).cumsum(1).cumsum(2)
    return s


def _inside(s, lo, hi):
    """Sum over [lo, hi) boxes (arrays per axis z, y, x), clipped to the array."""
    lo = [np.maximum(v, 0) for v in lo]
    hi = [np.minimum(v, n - 1) for v, n in zip(hi, s.shape)]
    out = 0
    for c in range(8):
        idx = tuple(hi[a] if (c >> a) & 1 else lo[a] for a in range(3))
        out = out + (1 if bin(c).count("1") % 2 else -1) * s[idx]
    return out


CASES = [((64, 64, 64), 0.02), ((64, 64, 64), 0.0005), ((37, 61, 50), 0.003), ((128, 10, 6), 0.01), ((1, 30, 33), 0.02),
         ((129, 127, 40), 0.0002), ((260, 16, 12), 0.001), ((2, 2, 2), 0.3), ((40, 40, 40), 0.0)]


@pytest.mark.parametrize("dtype", ["f32", "f16", "u8"])
@pytest.mark.parametrize("dims,density", CASES)
def test_boxes_are_free_and_layers_exact(dims, density, dtype):
    """Occupied bricks carry their voxels' occupancy and a voxel layer that is free as far as it
    says; free bricks a box without an occupied voxel (bricks without an entry count as occupied),
    as large as the free cube around them up to 7 bricks."""
    import torch
    from paper_2301_08068_amd import binding as B
    nx, ny, nz = dims
    rng = np.random.default_rng(nx * 131 + ny * 17 + nz)
    occ = rng.uniform(size=(nz, ny, nx)) < density
    occ[nz // 3, ny // 4:ny // 2, :] = density > 0              # a plate, so that slabs and layers matter
    val = np.where(occ, -0.1, 0.2).astype(np.float32)
    grid = {"f32": val, "f16": val.astype(np.float16).view(np.uint16), "u8": occ.astype(np.uint8)}[dtype]
    e = _entries(B, torch, grid, dtype).astype(np.int64)
    nb = np.array(e.shape)
    if e.size == 0:
        return
    full = [-(-n // 2) for n in occ.shape]
    pad = np.zeros([2 * n for n in full], bool)
    pad[:nz, :ny, :nx] = occ
    vox = pad.reshape(full[0], 2, full[1], 2, full[2], 2)
    mask = sum(vox[:, (b >> 2) & 1, :, (b >> 1) & 1, :, b & 1].astype(np.int64) << b for b in range(8))
    brick = np.ones(full, bool)                                  # bricks without an entry: never in a box
    brick[:nb[0], :nb[1], :nb[2]] = mask[:nb[0], :nb[1], :nb[2]] != 0
    mask = mask[:nb[0], :nb[1], :nb[2]]
    is_occ = (e & OCCUPIED) != 0
    assert np.array_equal(is_occ, mask != 0)
    assert np.array_equal(e[is_occ] & 0xff, mask[is_occ])
    z, y, x = np.nonzero(~is_occ)
    f = e[~is_occ]
    ext = [(f >> s & 31) // 2 for s in (10, 5, 0)]               # z, y, x
    assert all(np.all(v >= 1) for v in ext)
    assert not np.any(f & (1 | 1 << 5 | 1 << 10 | OCCUPIED))
    s = _sum(brick)
    c = (z, y, x)
    assert not np.any(_inside(s, [c[a] - ext[a] + 1 for a in range(3)], [c[a] + ext[a] for a in range(3)]))
    for k in range(1, 8):                                        # the cube of half extent k is free: so is the entry's
        free = _inside(s, [c[a] - k + 1 for a in range(3)], [c[a] + k for a in range(3)]) == 0
        assert np.all(np.minimum.reduce(ext)[free] >= k)
    assert np.all(np.maximum.reduce(ext) <= 15)
    if density == 0.0:
        # (40 voxels: 20 bricks; the centre's cube of 10 bricks reaches the surface all round)
        assert np.all(np.minimum.reduce(ext) >= 10)
    # layers of occupied bricks
    z, y, x = np.nonzero(is_occ)
    o = e[is_occ]
    axis, side, r = o >> AXIS & 3, o >> SIDE & 1, o >> EXTENT & 15
    none = axis == 3
    assert np.all(side[none] == 1)
    assert np.all(r[none] == 0) and np.all(r[~none] >= 1)
    for a in range(3):                                           # x, y, z; array axis 2 - a
        for sd in range(2):
            sub = [slice(None), slice(None)] * 3
            sub[2 * (2 - a) + 1] = sd
            layer = np.ones(full, bool)
            got = vox[tuple(sub)].any(axis=tuple(i for i in range(5) if i not in _brick_axes(2 - a)))
            layer[:nb[0], :nb[1], :nb[2]] = got[:nb[0], :nb[1], :nb[2]]
            k = (axis == a) & (side == sd)
            c, rr = (z[k], y[k], x[k]), r[k]
            d = [rr.copy(), rr.copy(), rr.copy()]
            d[2 - a] = np.ones_like(rr)
            assert not np.any(_inside(_sum(layer), [c[i] - d[i] + 1 for i in range(3)], [c[i] + d[i] for i in range(3)]))
            # a brick with a free layer says so
            has = ~got[:nb[0], :nb[1], :nb[2]][is_occ]
            assert not np.any(has & none)


@pytest.mark.parametrize("dtype", ["f32", "f16", "u8"])
@pytest.mark.parametrize("dims", [(64, 48, 40), (61, 47, 33), (128, 128, 96)])
def test_boxes_do_not_depend_on_the_source(dims, dtype):
    """The same entries from device memory at any address, from host memory, and in an arena that
    has no room for the upload's scratch."""
    import torch
    from paper_2301_08068_amd import binding as B
    nx, ny, nz = dims
    occ = np.random.default_rng(5).uniform(size=(nz, ny, nx)) < 0.01
    val = np.where(occ, -0.1, 0.2).astype(np.float32)
    grid = {"f32": val, "f16": val.astype(np.float16).view(np.uint16), "u8": occ.astype(np.uint8)}[dtype]
    ref = _entries(B, torch, grid, dtype)
    for source in ("offset", "host", "tight"):
        assert np.array_equal(_entries(B, torch, grid, dtype, source), ref), source


def _brick_axes(dropped):
    """Positions of the brick axes after indexing the sub-axis of `dropped` in a [b, 2, b, 2, b, 2] array."""
    out, pos = [], 0
    for i in range(3):
        out.append(pos)
        pos += 1 if i == dropped else 2
    return out


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("dims", [(63, 65, 67), (255, 8, 9), (1, 7, 5), (6, 301, 2), (64, 64, 65), (258, 3, 300)])
def test_the_whole_grid_is_copied(dims, dtype):
    """The resident grid equals the uploaded one, byte for byte, where bricks end at odd extents (the
    last layers of partial maps are copied apart from them)."""
    import torch
    from paper_2301_08068_amd import binding as B
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + ny + nz)
    val = rng.uniform(-0.3, 0.3, (nz, ny, nx)).astype(np.float32)
    grid = val if dtype == "f32" else val.astype(np.float16).view(np.uint16)
    arena = torch.zeros(ARENA, dtype=torch.uint8, device="cuda:0")
    ctx = B.rmpc_create(0, arena.data_ptr(), ARENA)
    try:
        dev = torch.from_numpy(np.ascontiguousarray(grid).view(np.uint8).reshape(-1)).to("cuda:0")
        before = arena.clone()
        B.rmpc_map_upload(ctx, nx, ny, nz, dtype, 0.1, (0.0, 0.0, 0.0), dev.data_ptr(), True)
        base = int(torch.nonzero(arena != before)[0]) // 256 * 256
        assert torch.equal(arena[base:base + dev.numel()], dev)
    finally:
        B.rmpc_destroy(ctx)


# words along y and along z: a few bricks wide in x, up to and past words of 64 bricks, odd extents
@pytest.mark.parametrize("dtype", ["f32", "f16", "u8"])
@pytest.mark.parametrize("dims,density", [((2, 128, 60), 0.002), ((1, 257, 9), 0.02), ((7, 131, 33), 0.003), ((3, 300, 258), 0.0005),
                                          ((6, 4, 150), 0.01), ((5, 3, 259), 0.01), ((1, 1, 384), 0.02), ((9, 34, 129), 0.0005),
                                          ((40, 300, 40), 0.0)])
def test_boxes_of_narrow_grids(dims, density, dtype):
    """As above, where the bit sets' words lie along another axis than x."""
    test_boxes_are_free_and_layers_exact(dims, density, dtype)


@pytest.mark.parametrize("dtype,shift", [("f32", 1), ("f32", 2), ("f32", 6), ("f16", 1), ("f16", 5)])
@pytest.mark.parametrize("dims", [(32, 20, 12), (31, 7, 9)])
def test_voxels_at_any_byte(dims, dtype, shift):
    """The caller's buffer may start anywhere: the resident grid and the rays' hits are those of an
    aligned one."""
    import torch
    from paper_2301_08068_amd import binding as B
    from paper_2301_08068_amd import workloads as W
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + shift)
    val = np.where(rng.uniform(size=(nz, ny, nx)) < 0.02, -0.1, rng.uniform(0.05, 0.3, (nz, ny, nx))).astype(np.float32)
    val[nz // 2, ny // 2, nx // 2] = 0.2
    grid = val if dtype == "f32" else W.encode_f16(val)
    raw = torch.from_numpy(np.ascontiguousarray(grid).view(np.uint8).reshape(-1))
    c = B.Context(0, arena_bytes=32 << 20)
    try:
        got = []
        for s in (0, shift):
            dev = torch.cat([torch.zeros(s, dtype=torch.uint8), raw]).to("cuda:0")
            mid = B.rmpc_map_upload(c.ptr, nx, ny, nz, dtype, 0.1, (0.0, 0.0, 0.0), dev.data_ptr() + s, True)
            x = (np.array([nx // 2, ny // 2, nz // 2]) + 0.4) * 0.1
            got.append(c.trace(mid, x, 2000, W.params("static", max_range=5.0, subvoxel=1)))
        for k in ("hit", "d", "visits"):
            assert np.array_equal(got[0][k], got[1][k]), k
    finally:
        c.close()
