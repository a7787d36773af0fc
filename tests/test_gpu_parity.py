"""GPU parity: the HIP path through the C ABI against the float64 oracle on the same seeded
inputs (tiny 64^3 map over 1000 states, the 400^3 paper-shaped map at 65536 rays, the
float16/uint8 encodings, LiDAR scans and edge cases)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_2301_08068_amd import workloads as W  # noqa: E402
from gpu_common import compare_query, compare_trace  # noqa: E402

P_TINY = W.params("static", max_range=5.0)
P_PAPER = W.params("static", max_range=10.0)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_08068_amd import binding
    c = binding.Context(0, arena_bytes=1 << 30)
    yield c
    c.close()


@pytest.fixture(scope="module")
def tiny(ctx, tiny_map):
    return ctx.upload(tiny_map.tsdf, tiny_map.voxel_m, tiny_map.origin_m, "f32"), \
        oracle.OracleMap.from_voxelmap(tiny_map)


@pytest.fixture(scope="module")
def paper(ctx, paper_map):
    return ctx.upload(paper_map.tsdf, paper_map.voxel_m, paper_map.origin_m, "f32"), \
        oracle.OracleMap.from_voxelmap(paper_map)


def test_direction_table_bit_equal(ctx):
    gpu = ctx.directions(65536)
    ref = oracle.directions(65536)
    assert np.array_equal(gpu.view(np.uint32), ref.view(np.uint32))


def test_tiny_trace_parity(ctx, tiny, tiny_map):
    mid, om = tiny
    dirs = oracle.directions(1024)
    n_same = n_flag = 0
    for seed in range(100, 300):
        x, _ = W.free_state(tiny_map, seed)
        g = ctx.trace(mid, x, 1024, P_TINY)
        o = oracle.trace(om, oracle.grid_start(om, x), dirs, P_TINY["max_range"])
        s, f = compare_trace(g, o, f"seed {seed}")
        n_same += s
        n_flag += f
    print(f"tiny trace: {n_same} / {200 * 1024} rays identical, {n_flag} flagged")


def test_tiny_query_parity_1000_states(ctx, tiny, tiny_map):
    mid, om = tiny
    dirs = oracle.directions(1024)
    n_ill = 0
    for seed in range(100, 1100):
        x, v = W.free_state(tiny_map, seed)
        g = ctx.query(mid, x, v, 1024, P_TINY)
        o = oracle.query(om, x, v, 1024, P_TINY, dirs=dirs)
        compare_query(g, o, f"seed {seed}")
        n_ill += bool(o["flags"] & oracle.Q_ILL)
    print(f"tiny queries: 1000 states, {n_ill} ILL")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1000, 4097, 65535, 65536])
def test_ragged_ray_counts(ctx, tiny, tiny_map, n):
    mid, om = tiny
    x, v = W.free_state(tiny_map, 100 + n % 7)
    g = ctx.query(mid, x, v, n, P_TINY)
    o = oracle.query(om, x, v, n, P_TINY)
    compare_query(g, o, f"n={n}")
    assert g["n_rays"] == n


def test_paper_map_parity_65536(ctx, paper, paper_map):
    mid, om = paper
    dirs = oracle.directions(65536)
    for seed in (200, 201, 202):
        x, v = W.free_state(paper_map, seed)
        g = ctx.trace(mid, x, 65536, P_PAPER)
        o = oracle.trace(om, oracle.grid_start(om, x), dirs, P_PAPER["max_range"], nthreads=8)
        compare_trace(g, o, f"paper seed {seed}")
        gq = ctx.query(mid, x, v, 65536, P_PAPER)
        oq = oracle.query(om, x, v, 65536, P_PAPER, dirs=dirs, nthreads=8)
        compare_query(gq, oq, f"paper seed {seed}")


@pytest.mark.parametrize("enc", ["f16", "u8"])
def test_encodings_match_f32(ctx, paper_map, enc):
    data = W.encode_f16(paper_map.tsdf) if enc == "f16" else W.encode_u8(paper_map.tsdf)
    mid_e = ctx.upload(data, paper_map.voxel_m, paper_map.origin_m, enc)
    om = oracle.OracleMap(data, paper_map.voxel_m, paper_map.origin_m, enc)
    try:
        x, v = W.free_state(paper_map, 200)
        g = ctx.trace(mid_e, x, 65536, P_PAPER)
        o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(65536), P_PAPER["max_range"],
                         nthreads=8)
        compare_trace(g, o, enc)
        compare_query(ctx.query(mid_e, x, v, 65536, P_PAPER),
                      oracle.query(om, x, v, 65536, P_PAPER, nthreads=8), enc)
    finally:
        ctx.release(mid_e)


def test_host_upload_equals_device_upload(ctx, tiny_map):
    a = ctx.upload(tiny_map.tsdf, tiny_map.voxel_m, tiny_map.origin_m, "f32", on_device=True)
    b = ctx.upload(tiny_map.tsdf, tiny_map.voxel_m, tiny_map.origin_m, "f32", on_device=False)
    x, v = W.free_state(tiny_map, 5)
    ra, rb = ctx.query(a, x, v, 4096, P_TINY), ctx.query(b, x, v, 4096, P_TINY)
    assert np.array_equal(ra["S"], rb["S"]) and np.array_equal(ra["f"], rb["f"])
    ctx.release(a)
    ctx.release(b)


def test_repeat_is_bitwise_identical(ctx, paper, paper_map):
    mid, _ = paper
    x, v = W.free_state(paper_map, 210)
    a = ctx.query(mid, x, v, 65536, P_PAPER)
    for _ in range(3):
        b = ctx.query(mid, x, v, 65536, P_PAPER)
        for k in ("S", "b", "f"):
            assert np.array_equal(a[k], b[k])


def test_zero_velocity_gives_exact_zero(ctx, tiny, tiny_map):
    mid, _ = tiny
    for seed in range(100, 120):
        x, _ = W.free_state(tiny_map, seed)
        r = ctx.query(mid, x, [0, 0, 0], 1024, P_TINY)
        assert np.all(r["S"] == 0) and np.all(r["b"] == 0) and np.all(r["f"] == 0)
        assert r["rank"] == 0 and r["n_contrib"] == 0


def test_in_collision_start(ctx, tiny, tiny_map):
    mid, om = tiny
    x = np.array([1.05, 1.05, 0.15])           # inside the floor slab
    g = ctx.query(mid, x, [0.3, 0.2, 1.0], 256, P_TINY)
    o = oracle.query(om, x, [0.3, 0.2, 1.0], 256, P_TINY)
    assert g["flags"] & 2 and o["flags"] & oracle.Q_IN_COLLISION
    compare_query(g, o, "in collision")
    t = ctx.trace(mid, x, 256, P_TINY)
    assert np.all(t["hit"] == 10 + 64 * (10 + 64 * 1)) and np.all(t["d"] == 0)


def test_scan_parity(ctx, tiny_map, paper_map):
    L = W.params("lidar")
    for vm, seed in ((tiny_map, 600), (paper_map, 601)):
        x, v = W.free_state(vm, seed)
        pts = W.synth_scan(vm, x, seed)
        g = ctx.scan_query(pts, v, L)
        o = oracle.scan(pts, v, L)
        compare_query(g, o, "scan")
        assert g["n_rays"] == pts.shape[0]


def test_scan_os0_scale_parity(ctx, paper_map):
    """A 128 x 2048 beam scan over a 90-degree vertical field of view (262,144 points, the
    size of the largest common spinning LiDAR frames)."""
    L = W.params("lidar")
    for seed in (610, 611):
        x, v = W.free_state(paper_map, seed)
        pts = W.synth_scan(paper_map, x, seed, n_elev=128, n_azim=2048, fov_deg=90.0)
        g = ctx.scan_query(pts, v, L)
        o = oracle.scan(pts, v, L)
        compare_query(g, o, f"os0 scan seed {seed}")
        assert g["n_rays"] == pts.shape[0] == 262144 and g["n_hit"] == o["n_hit"]


@pytest.mark.parametrize("n", [1001, 262145, 300001, 600000])
def test_scan_sizes_across_point_batches(ctx, n):
    """Scans whose threads take their points in several batches of eight with a ragged last one
    (128 blocks x 256 threads x 8 points = 262,144 points per batch round): random points within
    12 m, some dropouts (zeros) and non-finite entries."""
    L = W.params("lidar")
    rng = np.random.default_rng(n)
    pts = (rng.normal(size=(n, 3)) * rng.uniform(0.05, 12.0, size=(n, 1)) /
           np.sqrt(3.0)).astype(np.float32)
    pts[rng.uniform(size=n) < 0.1] = 0.0
    pts[rng.integers(0, n, size=3), rng.integers(0, 3, size=3)] = np.nan
    v = [1.5, -0.5, 0.25]
    g = ctx.scan_query(pts, v, L)
    o = oracle.scan(pts, v, L)
    compare_query(g, o, f"scan of {n} points")
    assert g["n_rays"] == n and g["n_hit"] == o["n_hit"]


def test_scan_reproduces_grid_query(ctx, tiny, tiny_map):
    mid, om = tiny
    dirs = oracle.directions(1024)
    for seed in range(100, 110):
        x, v = W.free_state(tiny_map, seed)
        tr = oracle.trace(om, oracle.grid_start(om, x), dirs, 5.0)
        hit = tr["hit"] >= 0
        pts = (dirs[hit].astype(np.float64) * tr["d"][hit, None]).astype(np.float32)
        q = ctx.query(mid, x, v, 1024, P_TINY)
        s = ctx.scan_query(pts, v, dict(P_TINY, min_range=1e-9))
        sS = max(np.abs(q["S"]).max(), 1e-300)
        assert np.max(np.abs(s["S"] - q["S"])) <= 1e-4 * sS
        assert np.max(np.abs(s["b"] - q["b"])) <= 1e-4 * max(np.abs(q["b"]).max(), 1e-300)


def test_scan_edge_cases(ctx):
    L = W.params("lidar")
    empty = ctx.scan_query(np.zeros((0, 3), np.float32), [1, 0, 0], L)
    assert empty["n_hit"] == 0 and np.all(empty["f"] == 0)
    bad = np.array([[0, 0, 0], [np.nan, 1, 1], [np.inf, 0, 0], [0.05, 0, 0], [0.5, 0, 0]], np.float32)
    r = ctx.scan_query(bad, [1, 0, 0], L)
    o = oracle.scan(bad, [1, 0, 0], L)
    assert r["n_hit"] == 1 == o["n_hit"]
    compare_query(r, o, "scan edge")


def test_errors_are_reported(ctx, tiny, tiny_map):
    from paper_2301_08068_amd import binding as B
    mid, _ = tiny
    with pytest.raises(B.RmpcError) as e:
        ctx.query(mid, [-1.0, 1, 1], [0, 0, 0], 64, P_TINY)
    assert e.value.status == B.RMPC_E_OUT_OF_BOUNDS
    for bad in ([np.nan, 1, 1], [np.inf, 1, 1]):
        with pytest.raises(B.RmpcError) as e:
            ctx.query(mid, bad, [0, 0, 0], 64, P_TINY)
        assert e.value.status == B.RMPC_E_INVALID
    for n in (0, 65537, -3):
        with pytest.raises(B.RmpcError) as e:
            ctx.query(mid, [1, 1, 1], [0, 0, 0], n, P_TINY)
        assert e.value.status == B.RMPC_E_INVALID
    with pytest.raises(B.RmpcError) as e:
        ctx.query(12345, [1, 1, 1], [0, 0, 0], 64, P_TINY)
    assert e.value.status == B.RMPC_E_NOMAP
    with pytest.raises(B.RmpcError) as e:
        ctx.query(mid, [1, 1, 1], [0, 0, 0], 64, dict(P_TINY, nu_rep=0.0))
    assert e.value.status == B.RMPC_E_INVALID
    with pytest.raises(B.RmpcError) as e:
        ctx.upload(np.zeros((4, 4, 4), np.float32), 0.0, (0, 0, 0))
    assert e.value.status == B.RMPC_E_INVALID


@pytest.mark.parametrize("crop", [(0, 61, 3, 70, 1, 64), (5, 64, 0, 63, 0, 57), (0, 13, 0, 64, 0, 6)])
def test_partial_cells_parity(ctx, tiny_map, crop):
    """Grids whose sides are not multiples of 8 (partial cells are walked voxel by voxel) and a
    grid thinner than one cell (no cell summaries at all): every ray as the oracle's."""
    x0, x1, y0, y1, z0, z1 = crop
    t = np.ascontiguousarray(tiny_map.tsdf[z0:z1, y0:y1, x0:x1])
    org = tiny_map.origin_m + np.array([x0, y0, z0]) * tiny_map.voxel_m
    mid = ctx.upload(t, tiny_map.voxel_m, org, "f32")
    om = oracle.OracleMap(t, tiny_map.voxel_m, org, "f32")
    try:
        rng = np.random.default_rng(sum(crop))
        done = 0
        while done < 6:
            x = org + rng.uniform(0.0, 1.0, 3) * np.array(t.shape[::-1]) * tiny_map.voxel_m
            gi = np.floor((x - org) / tiny_map.voxel_m).astype(int)
            if t[gi[2], gi[1], gi[0]] <= 0:
                continue
            v = rng.normal(size=3)
            g = ctx.trace(mid, x, 4096, P_TINY)
            o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(4096), P_TINY["max_range"])
            compare_trace(g, o, f"crop {t.shape} state {done}")
            compare_query(ctx.query(mid, x, v, 4096, P_TINY), oracle.query(om, x, v, 4096, P_TINY),
                          f"crop {t.shape} state {done}")
            done += 1
    finally:
        ctx.release(mid)


def test_corner_starts_and_cell_face_ranges(ctx, tiny, tiny_map):
    """Starts on voxel and cell corners and ranges that end exactly on cell faces."""
    mid, om = tiny
    for g in ((16.0, 16.0, 16.0), (8.0, 24.0, 40.0), (17.0, 33.0, 9.5), (31.5, 32.0, 32.0)):
        x = tiny_map.origin_m + np.array(g) * tiny_map.voxel_m
        gi = np.floor(g).astype(int)
        if tiny_map.tsdf[gi[2], gi[1], gi[0]] <= 0:
            continue
        for rmax in (0.8, 1.6):
            P = dict(P_TINY, max_range=rmax)
            gt = ctx.trace(mid, x, 4096, P)
            o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(4096), rmax)
            compare_trace(gt, o, f"corner {g} range {rmax}")


@pytest.mark.parametrize("density", [0.0, 0.02, 0.15])
def test_random_occupancy_parity(ctx, density):
    """Random occupancy on an odd-sized 61 x 66 x 59 grid.  With 2 % of the voxels occupied
    nearly every 8^3 cell is occupied while most 2^3 bricks are free, so walks go down from
    cells to bricks and back up all the time; at 15 % few bricks are free; an empty grid is
    walked at the coarsest level up to its edge (and its partial bricks and cells voxel by
    voxel).  Every ray as the oracle's, for lookahead 4, 8 and 16."""
    from paper_2301_08068_amd import binding as B
    rng = np.random.default_rng(int(density * 1000) + 7)
    shape = (59, 66, 61)                       # z, y, x
    t = np.where(rng.uniform(size=shape) < density, -0.05, 0.05).astype(np.float32)
    h, org = 0.1, np.array([-1.0, 0.5, 2.0])
    mid = ctx.upload(t, h, org, "f32")
    om = oracle.OracleMap(t, h, org, "f32")
    saved = ctx.config(B.CONFIG_QUERY)
    try:
        for K in (4, 8, 16):
            ctx.config(B.CONFIG_QUERY, lookahead=K)
            for s in range(2):
                while True:
                    gi = rng.integers(0, shape[::-1])          # x, y, z
                    if t[gi[2], gi[1], gi[0]] > 0:
                        break
                x = org + (gi + rng.uniform(0.05, 0.95, 3)) * h
                for rmax in (2.5, 8.0):
                    P = dict(P_TINY, max_range=rmax)
                    g = ctx.trace(mid, x, 4096, P)
                    o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(4096), rmax)
                    compare_trace(g, o, f"density {density} lookahead {K} state {s} range {rmax}")
    finally:
        ctx.config(B.CONFIG_QUERY, **saved)
        ctx.release(mid)


def test_long_walks_parity(ctx):
    """A 2500 x 36 x 10 grid with sparse obstacles and a 130 m range (2600 voxels): rays along
    the long axis walk thousands of voxels split into 8 and 16 segments, so segment ends lie far
    along the ray, where float32 crossing parameters carry their largest absolute error."""
    from paper_2301_08068_amd import binding as B
    rng = np.random.default_rng(11)
    shape = (10, 36, 2500)
    t = np.where(rng.uniform(size=shape) < 0.0004, -0.05, 0.05).astype(np.float32)
    h, org = 0.05, np.zeros(3)
    mid = ctx.upload(t, h, org, "f32")
    om = oracle.OracleMap(t, h, org, "f32")
    saved = ctx.config(B.CONFIG_QUERY)
    P = dict(P_TINY, max_range=130.0)
    try:
        for s in range(3):
            while True:
                gi = np.array([rng.integers(0, 40), rng.integers(0, 36), rng.integers(0, 10)])
                if t[gi[2], gi[1], gi[0]] > 0:
                    break
            x = org + (gi + rng.uniform(0.05, 0.95, 3)) * h
            o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(8192), P["max_range"])
            for lt in (17, 20):
                ctx.config(B.CONFIG_QUERY, lookahead=8, lane_target_log2=lt)
                compare_trace(ctx.trace(mid, x, 8192, P), o, f"long state {s} lane target 2^{lt}")
    finally:
        ctx.config(B.CONFIG_QUERY, **saved)
        ctx.release(mid)


@pytest.mark.parametrize("enc", ["f32", "f16"])
def test_special_values_occupancy(ctx, enc):
    """Maps holding +-0, +-inf, NaNs of both signs and subnormals of both signs: a voxel is
    occupied exactly when its value compares <= 0 (NaN free, -0 occupied, a positive subnormal
    free), in the walk and in the cell and brick summaries alike."""
    rng = np.random.default_rng(31 if enc == "f32" else 32)
    shape = (36, 40, 48)
    if enc == "f32":
        specials = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, -np.nan, 1e-45, -1e-45, 1.0, -1.0],
                            np.float32).view(np.uint32)
        free = np.float32(0.05).view(np.uint32)
        t = np.full(shape, free, np.uint32)
    else:
        specials = np.array([0x0000, 0x8000, 0x7c00, 0xfc00, 0x7e00, 0xfe00, 0x0001, 0x8001, 0x3c00, 0xbc00],
                            np.uint16)
        t = np.full(shape, 0x2a66, np.uint16)                   # binary16 0.05
    mask = rng.uniform(size=shape) < 0.03
    t[mask] = rng.choice(specials, size=int(mask.sum()))
    data = t.view(np.float32) if enc == "f32" else t
    h, org = 0.1, np.zeros(3)
    mid = ctx.upload(data, h, org, enc)
    om = oracle.OracleMap(data, h, org, enc)
    try:
        for s in range(4):
            while True:
                gi = rng.integers(0, shape[::-1])
                v = data[gi[2], gi[1], gi[0]]
                if (enc == "f32" and v > 0) or (enc == "f16" and int(v) in (0x2a66, 0x3c00, 0x7c00)):
                    break
            x = org + (gi + rng.uniform(0.05, 0.95, 3)) * h
            P = dict(P_TINY, max_range=6.0)
            o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(4096), P["max_range"])
            compare_trace(ctx.trace(mid, x, 4096, P), o, f"{enc} specials state {s}")
    finally:
        ctx.release(mid)


@pytest.mark.parametrize("n,lanes_log2", [(16, 10), (60097, 16), (65536, 16), (60097, 17), (65536, 17), (65536, 18), (65536, 20)])
def test_reduction_over_few_and_many_blocks(ctx, tiny, tiny_map, n, lanes_log2):
    """1, 235, 256, 470, 512, 1,024 and 4,096 blocks: the last block's passes of 256 rows with and
    without a rest."""
    mid, om = tiny
    x, v = W.free_state(tiny_map, 117)
    before = ctx.config(0)
    try:
        ctx.config(0, lane_target_log2=lanes_log2)
        g = ctx.query(mid, x, v, n, P_TINY)
    finally:
        ctx.config(0, **before)
    compare_query(g, oracle.query(om, x, v, n, P_TINY, nthreads=8), f"n={n}")
