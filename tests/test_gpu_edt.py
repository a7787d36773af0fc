"""GPU exact distance transform (rmpc_edt) against the oracle's: every voxel bit for bit on the
tiny map in all three encodings and on ragged random grids; sampled voxels of the 400^3 map
against brute force over all its occupied voxels; empty and full grids."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_2301_08068_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_08068_amd import binding
    c = binding.Context(0, arena_bytes=1 << 30)
    yield c
    c.close()


def _gpu_edt(ctx, data, h, enc):
    mid = ctx.upload(data, h, np.zeros(3), enc)
    try:
        return ctx.edt(mid, data.shape).cpu().numpy()
    finally:
        ctx.release(mid)


@pytest.mark.parametrize("enc", ["f32", "f16", "u8"])
def test_tiny_map_bitwise(ctx, tiny_map, enc):
    data = {"f32": tiny_map.tsdf, "f16": W.encode_f16(tiny_map.tsdf), "u8": W.encode_u8(tiny_map.tsdf)}[enc]
    g = _gpu_edt(ctx, data, tiny_map.voxel_m, enc)
    o = oracle.edt(oracle.OracleMap(data, tiny_map.voxel_m, tiny_map.origin_m, enc))
    assert np.array_equal(g, o)


# line groups of the y and z passes: 64 lines of 23 (one partial group), 32 of 300, 16 of 1,000
# with a ragged last group (37 = 2 x 16 + 5), and single-element lines
@pytest.mark.parametrize("shape,p", [((37, 23, 51), 0.002), ((5, 300, 7), 0.01), ((64, 1, 130), 0.05),
                                     ((3, 1000, 37), 0.003), ((1000, 2, 70), 0.002)])
def test_ragged_random_grids(ctx, shape, p):
    rng = np.random.default_rng(sum(shape))
    occ = rng.uniform(size=shape) < p
    occ[0, 0, 0] = True
    t = np.where(occ, -0.05, 0.3).astype(np.float32)
    g = _gpu_edt(ctx, t, 0.1, "f32")
    assert np.array_equal(g, oracle.edt(oracle.OracleMap(t, 0.1, np.zeros(3), "f32")))


def test_longest_lines(ctx):
    """y and z lines of 4,096 voxels (the largest extent a map may have): two lines per group of
    the y and z passes; every voxel against the oracle."""
    rng = np.random.default_rng(7)
    for shape in ((1, 4096, 3), (4096, 1, 3)):
        t = np.where(rng.uniform(size=shape) < 0.001, -0.05, 0.3).astype(np.float32)
        t.reshape(-1)[1234] = -0.05
        g = _gpu_edt(ctx, t, 0.1, "f32")
        assert np.array_equal(g, oracle.edt(oracle.OracleMap(t, 0.1, np.zeros(3), "f32"))), shape


def test_empty_and_full(ctx):
    free = np.full((9, 10, 11), 0.3, np.float32)
    assert np.all(_gpu_edt(ctx, free, 0.1, "f32") == -1)
    assert np.all(_gpu_edt(ctx, -free, 0.1, "f32") == 0)


def test_paper_map_sampled(ctx, paper_map):
    g = _gpu_edt(ctx, paper_map.tsdf, paper_map.voxel_m, "f32")
    occ = paper_map.tsdf <= 0
    assert np.all(g[occ] == 0) and np.all(g[~occ] > 0)
    pts = np.argwhere(occ).astype(np.int64)               # (k, j, i)
    rng = np.random.default_rng(12)
    for _ in range(48):
        k, j, i = (int(v) for v in rng.integers(0, 400, size=3))
        best = int(np.min((pts[:, 0] - k) ** 2 + (pts[:, 1] - j) ** 2 + (pts[:, 2] - i) ** 2))
        assert g[k, j, i] == best, (k, j, i)


def test_esdf_policy_matches_oracle(ctx, tiny_map):
    """The single-lookup ESDF policy at many states of the tiny map: counts and flags exact,
    sums and the resolved acceleration to 1e-9 of their size (float64 on both sides; only the
    exp and log1p of the policy round differently)."""
    from paper_2301_08068_amd import binding as B
    mid = ctx.upload(tiny_map.tsdf, tiny_map.voxel_m, tiny_map.origin_m, "f32")
    om = oracle.OracleMap.from_voxelmap(tiny_map)
    p = W.params("static")
    try:
        sq = ctx.edt(mid, tiny_map.tsdf.shape)
        osq = oracle.edt(om)
        n_contrib = 0
        for seed in range(900, 1000):
            x, v = W.free_state(tiny_map, seed)
            g = ctx.esdf_query(mid, sq, x, v, p)
            o = oracle.esdf_query(om, osq, x, v, p)
            for k in ("n_hit", "n_contrib", "flags", "rank"):
                assert g[k] == o[k], (seed, k, g[k], o[k])
            for k in ("S", "b", "f"):
                scale = max(np.abs(o[k]).max(), 1e-300)
                assert np.abs(g[k] - o[k]).max() <= 1e-9 * scale, (seed, k, g[k], o[k])
            n_contrib += o["n_contrib"]
        assert n_contrib > 20
        with pytest.raises(B.RmpcError) as e:
            ctx.esdf_query(mid, sq, [-1.0, 0.5, 0.5], [0, 0, 0], p)
        assert e.value.status == B.RMPC_E_OUT_OF_BOUNDS
    finally:
        ctx.release(mid)


@pytest.mark.parametrize("room", [True, False])
@pytest.mark.parametrize("enc", ["f32", "f16", "u8"])
@pytest.mark.parametrize("shape,p", [((64, 65, 33), 0.003), ((63, 128, 32), 0.0005), ((129, 66, 31), 0.002),
                                     ((2, 257, 65), 0.002), ((300, 3, 40), 0.2)])
def test_chunk_and_strip_edges(shape, p, enc, room):
    """Lines of one element less, as many and one more than the passes' chunks of 64, strips of 32
    lines with and without a rest, in an arena with room for the rows' words and in a full one (the
    row distances then pass through the field)."""
    from paper_2301_08068_amd import binding
    rng = np.random.default_rng(sum(shape))
    occ = rng.uniform(size=shape) < p
    occ[-1, -1, -1] = True
    t = np.where(occ, -0.05, 0.3).astype(np.float32)
    data = {"f32": t, "f16": W.encode_f16(t), "u8": W.encode_u8(t)}[enc]
    c = binding.Context(0, arena_bytes=24 << 20)
    try:
        mid = c.upload(data, 0.1, np.zeros(3), enc)
        n = 0 if room else 1 << 15
        while n:
            try:
                c.upload(np.zeros((n, 1, 256), np.uint8), 0.1, np.zeros(3), "u8") if n <= 4096 else \
                    c.upload(np.zeros((4096, 1, n >> 4), np.uint8), 0.1, np.zeros(3), "u8")
            except binding.RmpcError as e:
                assert e.status == binding.RMPC_E_NOMEM
                n >>= 1
        g = c.edt(mid, shape).cpu().numpy()
    finally:
        c.close()
    assert np.array_equal(g, oracle.edt(oracle.OracleMap(data, 0.1, np.zeros(3), enc)))


# (one occupied voxel in a corner) the farthest voxel at 255, at 256 and beyond; strips without any
# occupied voxel beside others; a single row, column and voxel
@pytest.mark.parametrize("shape", [(1, 256, 1), (1, 257, 1), (256, 1, 3), (257, 2, 3), (3, 2, 256), (3, 2, 257),
                                   (2, 300, 70), (5, 3, 600), (181, 181, 2), (182, 182, 2), (1, 1, 1), (3, 2, 1)])
@pytest.mark.parametrize("at", [0, -1])
def test_distances_around_the_narrow_limit(ctx, shape, at):
    t = np.full(shape, 0.3, np.float32)
    t.reshape(-1)[at] = -0.05
    g = _gpu_edt(ctx, t, 0.1, "f32")
    assert np.array_equal(g, oracle.edt(oracle.OracleMap(t, 0.1, np.zeros(3), "f32")))


@pytest.mark.parametrize("n", [207, 208, 209, 831, 832, 833, 1665, 4000, 4001])
def test_strip_widths(ctx, n):
    """Lines of the lengths at which the strips narrow, along y and along z, with a rest of lines."""
    rng = np.random.default_rng(n)
    for shape in ((2, n, 35), (n, 2, 35)):
        t = np.where(rng.uniform(size=shape) < 0.002, -0.05, 0.3).astype(np.float32)
        t.reshape(-1)[n] = -0.05
        g = _gpu_edt(ctx, t, 0.1, "f32")
        assert np.array_equal(g, oracle.edt(oracle.OracleMap(t, 0.1, np.zeros(3), "f32")))


@pytest.mark.parametrize("shape", [(4, 5, 6), (1, 5, 6), (4, 1, 1), (1, 1, 1)])
def test_esdf_neighbours_at_the_grid_edges(ctx, shape):
    """Every voxel of a tiny grid, its neighbours clamped at the edges; alternating with a map
    without an occupied voxel (zero sums).  Tolerance as above."""
    rng = np.random.default_rng(sum(shape))
    p = W.params("static")
    for occupied in (True, False):
        t = np.full(shape, 0.3, np.float32)
        if occupied:
            t.reshape(-1)[rng.integers(t.size)] = -0.1
        om = oracle.OracleMap(t, 0.5, np.zeros(3), "f32")
        mid = ctx.upload(t, 0.5, np.zeros(3), "f32")
        try:
            sq, osq = ctx.edt(mid, shape), oracle.edt(om)
            for z, y, x in np.ndindex(shape):
                at, v = (np.array([x, y, z]) + 0.5) * 0.5, rng.normal(0.0, 1.0, 3)
                g, o = ctx.esdf_query(mid, sq, at, v, p), oracle.esdf_query(om, osq, at, v, p)
                assert (g["n_rays"], g["n_tie"], g["visits"]) == (1, 0, 0)
                for k in ("n_hit", "n_contrib", "flags", "rank"):
                    assert g[k] == o[k], (x, y, z, k, g[k], o[k])
                for k in ("S", "b", "f"):
                    assert np.abs(g[k] - o[k]).max() <= 1e-9 * max(np.abs(o[k]).max(), 1e-300), (x, y, z, k)
        finally:
            ctx.release(mid)


# more strips than the GPU holds at once (the last pass has 15,040 and 24,000 blocks), so that blocks
# start, load and search while others give the narrow passes up
@pytest.mark.parametrize("shape,at", [((300, 160, 1500), [(0, 0, 0)]), ((1000, 48, 4000), [(0, 0, 0), (999, 47, 2000)])])
def test_given_up_while_other_blocks_run(ctx, shape, at):
    """Too far for the narrow passes: the distance to a few voxels, from its definition."""
    occ = np.zeros(shape, np.uint8)
    axes = [torch.arange(n, dtype=torch.int32, device="cuda:0") for n in shape]
    want = None
    for c in at:
        occ[c] = 1
        z, y, x = ((a - i) ** 2 for a, i in zip(axes, c))
        d = z[:, None, None] + y[None, :, None] + x[None, None, :]
        want = d if want is None else torch.minimum(want, d)
    mid = ctx.upload(occ, 0.1, np.zeros(3), "u8")
    try:
        assert torch.equal(ctx.edt(mid, shape), want)
    finally:
        ctx.release(mid)


# (diagonals around the narrow limit, 255^2 + 255^2 ... : 65,534, 65,536 and beyond) no occupied voxel,
# one in a corner, all
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 3, 5), (8, 8, 8), (64, 64, 64), (2, 1, 256), (148, 149, 149), (149, 149, 149),
                                   (16, 8, 256), (1, 1, 257)])
def test_small_grids_without_a_watch(ctx, shape):
    for fill in (0, 1, 2):
        occ = np.full(shape, fill == 2, np.uint8)
        occ.reshape(-1)[-1] |= fill == 1
        z, y, x = (np.arange(n - 1, -1, -1) ** 2 for n in shape)
        one = z[:, None, None] + y[None, :, None] + x[None, None, :]
        want = {0: np.full(shape, -1), 1: one, 2: np.zeros(shape)}[fill]
        assert np.array_equal(_gpu_edt(ctx, occ, 0.1, "u8"), want), fill


@pytest.mark.parametrize("enc", ["f32", "u8"])
@pytest.mark.parametrize("shape,p", [((64, 65, 33), 0.003), ((129, 66, 31), 0.002), ((2, 257, 65), 0.002), ((300, 3, 40), 0.2),
                                     ((3, 2, 257), 0.0), ((182, 182, 2), 0.0)])
def test_room_for_the_flags_alone(shape, p, enc):
    """An arena with 256 bytes left: the narrow passes with the row distances through the field (and
    the wide ones after them where a distance reaches 256)."""
    from paper_2301_08068_amd import binding
    rng = np.random.default_rng(sum(shape))
    occ = rng.uniform(size=shape) < p
    occ[-1, -1, -1] = True
    t = np.where(occ, -0.05, 0.3).astype(np.float32)
    data = t if enc == "f32" else W.encode_u8(t)
    c = binding.Context(0, arena_bytes=24 << 20)
    try:
        mid = c.upload(data, 0.1, np.zeros(3), enc)
        assert binding.rmpc_map_footprint(256, 1, 1, "u8", 0.1, (0, 0, 0)) == 256
        held = c.upload(np.zeros((1, 1, 256), np.uint8), 0.1, np.zeros(3), "u8")
        for dims in ((4096, 1, 256), (256, 1, 256), (16, 1, 256), (1, 1, 256)):
            while True:
                try:
                    c.upload(np.zeros(dims, np.uint8), 0.1, np.zeros(3), "u8")
                except binding.RmpcError as e:
                    assert e.status == binding.RMPC_E_NOMEM
                    break
        c.release(held)
        g = c.edt(mid, shape).cpu().numpy()
    finally:
        c.close()
    assert np.array_equal(g, oracle.edt(oracle.OracleMap(data, 0.1, np.zeros(3), enc)))
