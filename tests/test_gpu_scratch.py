"""Uploads that get no scratch (a full arena on a full device): maps walked by narrower boxes, or by
the block table, give the same hits, distances, visits and sums."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from gpu_common import compare_trace  # noqa: E402
from paper_2301_08068_amd import workloads as W  # noqa: E402

P = W.params("static", max_range=5.0)


@pytest.fixture()
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_08068_amd import binding
    c = binding.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


def _limit(c, n):
    from paper_2301_08068_amd import binding
    binding._lib.rmpc_internal_scratch_limit(C.c_void_p(c.ptr), C.c_size_t(n))


def _same_query(a, b):
    for k in ("f", "S", "b", "lam"):
        assert np.array_equal(a[k], b[k]), k
    for k in ("rank", "n_hit", "n_contrib", "visits"):
        assert a[k] == b[k], k


# even extents, odd ones (an odd last layer without entries for some types), walls of bricks at the
# edges, a single layer, fewer bricks than a box reaches
@pytest.mark.parametrize("on_device", [True, False])
@pytest.mark.parametrize("enc", ["f32", "f16", "u8"])
@pytest.mark.parametrize("dims,p", [((64, 48, 40), 0.003), ((61, 47, 33), 0.003), ((63, 1, 65), 0.01), ((5, 3, 4), 0.05),
                                    ((1, 1, 1), 0.0), ((40, 41, 39), 0.0)])
def test_dense_without_scratch(ctx, dims, p, enc, on_device):
    nx, ny, nz = dims
    rng = np.random.default_rng(sum(dims))
    t = np.where(rng.uniform(size=(nz, ny, nx)) < p, -0.05, 0.3).astype(np.float32)
    data = {"f32": t, "f16": W.encode_f16(t), "u8": W.encode_u8(t)}[enc]
    om = oracle.OracleMap(data, 0.1, np.zeros(3), enc)
    full = ctx.upload(data, 0.1, np.zeros(3), enc, on_device=on_device)
    _limit(ctx, 0)
    mid = ctx.upload(data, 0.1, np.zeros(3), enc, on_device=on_device)
    free = np.argwhere(t > 0)
    for at in free[rng.integers(len(free), size=4)]:
        x = (at[::-1] + rng.uniform(0.1, 0.9, 3)) * 0.1
        o = oracle.trace(om, oracle.grid_start(om, x), oracle.directions(4096), P["max_range"])
        compare_trace(ctx.trace(mid, x, 4096, P), o, f"{dims} {enc}")
        v = rng.normal(size=3)
        _same_query(ctx.query(mid, x, v, 1000, P), ctx.query(full, x, v, 1000, P))
    assert torch.equal(ctx.edt(mid, t.shape), ctx.edt(full, t.shape))


@pytest.mark.parametrize("enc,subvoxel", [("f32", 0), ("f16", 1), ("u8", 0)])
def test_sparse_without_scratch(ctx, tiny_map, enc, subvoxel):
    """Walked by the table instead of the index."""
    sm = W.sparse_from_dense(tiny_map, offset_blocks=(-3, 2, 5), keep_free=0.3, seed=4)
    data = {"f32": sm.values, "f16": W.encode_f16(sm.values), "u8": W.encode_u8(sm.values)}[enc]
    full = ctx.upload_sparse(sm.coords, data, sm.voxel_m, sm.origin_m, enc)
    _limit(ctx, 0)
    mid = ctx.upload_sparse(sm.coords, data, sm.voxel_m, sm.origin_m, enc)
    p = dict(P, subvoxel=subvoxel)
    for seed in range(6):
        x, v = W.free_state(tiny_map, seed)
        x = x + np.array([-3, 2, 5]) * 8 * sm.voxel_m + (sm.origin_m - tiny_map.origin_m)
        a, b = ctx.trace(mid, x, 4096, p), ctx.trace(full, x, 4096, p)
        for k in ("hit", "d", "visits"):
            assert np.array_equal(a[k], b[k]), (seed, k)
        _same_query(ctx.query(mid, x, v, 4096, p), ctx.query(full, x, v, 4096, p))
        if not subvoxel:
            q = [dict(kind="map", map_id=m, n=700, x=x, v=v) for m in (mid, full)]
            _same_query(*ctx.query_batch(q, p, None))


@pytest.mark.parametrize("short", [0, 1])
def test_scratch_is_all_or_nothing(ctx, short):
    """A limit of exactly the need, and one byte less."""
    t = np.full((40, 40, 40), 0.3, np.float32)
    t[30] = -0.1
    need = 20 * 20 * 20 // 256 * 256 + 256 + 8 * 52 * 20 * 20          # masks (20 bytes a row), 52 bit sets of a word a row
    _limit(ctx, need - short)
    mid = ctx.upload(t, 0.1, np.zeros(3), "f32")
    om = oracle.OracleMap(t, 0.1, np.zeros(3), "f32")
    x = np.array([2.03, 1.97, 1.01])
    compare_trace(ctx.trace(mid, x, 4096, P), oracle.trace(om, oracle.grid_start(om, x), oracle.directions(4096), P["max_range"]))


@pytest.mark.parametrize("enc,source", [("f32", "device"), ("f16", "offset"), ("u8", "device"), ("u8", "host")])
@pytest.mark.parametrize("dims,p", [((64, 64, 64), 0.0005), ((61, 47, 33), 0.001), ((63, 1, 65), 0.01), ((130, 3, 4), 0.003), ((40, 40, 40), 0.0)])
def test_boxes_without_scratch_are_wide(monkeypatch, dims, p, enc, source):
    """A free brick's box is the widest free cube of half extent 1, 2, 3, 5 or 9 around it (bricks
    without an entry count as occupied, those outside the grid as free); an occupied brick's entry holds
    its voxels and no layer."""
    import test_gpu_boxes as T
    from paper_2301_08068_amd import binding as B
    create = B.rmpc_create

    def limited(*a):
        ctx = create(*a)
        B._lib.rmpc_internal_scratch_limit(C.c_void_p(ctx), C.c_size_t(0))
        return ctx

    monkeypatch.setattr(B, "rmpc_create", limited)
    nx, ny, nz = dims
    occ = np.random.default_rng(sum(dims)).uniform(size=(nz, ny, nx)) < p
    t = np.where(occ, -0.1, 0.2).astype(np.float32)
    grid = {"f32": t, "f16": W.encode_f16(t), "u8": W.encode_u8(t)}[enc]
    e = T._entries(B, torch, grid, enc, source).astype(np.int64)
    full = [-(-n // 2) for n in occ.shape]
    pad = np.zeros([2 * n for n in full], bool)
    pad[:nz, :ny, :nx] = occ
    vox = pad.reshape(full[0], 2, full[1], 2, full[2], 2)
    mask = sum(vox[:, (b >> 2) & 1, :, (b >> 1) & 1, :, b & 1].astype(np.int64) << b for b in range(8))
    nb = e.shape
    brick = np.ones(full, bool)
    brick[:nb[0], :nb[1], :nb[2]] = mask[:nb[0], :nb[1], :nb[2]] != 0
    mask = mask[:nb[0], :nb[1], :nb[2]]
    c = np.nonzero(mask == 0)
    want = np.ones(len(c[0]), np.int64)
    for k in (2, 3, 5, 9):
        want[T._inside(T._sum(brick), [v - k + 1 for v in c], [v + k for v in c]) == 0] = k
    assert np.array_equal(e[mask == 0], 2 * want * (1 | 1 << 5 | 1 << 10))
    assert np.array_equal(e[mask != 0], mask[mask != 0] | T.OCCUPIED | 1 << T.SIDE | 3 << T.AXIS)


def test_sparse_scratch_comes_from_the_arena(tiny_map):
    """With room, the upload of a sparse map takes its scratch from the arena (bytes past the map's own
    change); in an arena that has just the map's own room it is uploaded all the same, with equal hits."""
    from paper_2301_08068_amd import binding as B
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sm = W.sparse_from_dense(tiny_map, keep_free=0.3, seed=4)
    n, size = len(sm.coords), 48 << 20
    cap = 1024
    while cap < 16 * n:
        cap *= 2
    own = sum(-(-b // 256) * 256 for b in (16 * cap, 64 * n, 4 * 512 * n))
    arena = torch.zeros(size, dtype=torch.uint8, device="cuda:0")
    ctx = B.rmpc_create(0, arena.data_ptr(), size)
    vals = torch.from_numpy(np.ascontiguousarray(sm.values, np.float32)).to("cuda:0")
    x, _ = W.free_state(tiny_map, 3)

    def upload():
        return B.rmpc_sparse_map_upload(ctx, sm.coords, vals.data_ptr(), n, "f32", sm.voxel_m, sm.origin_m, True, free_value=0.3)

    def trace(mid):
        hit, d = torch.empty(2000, dtype=torch.int32, device="cuda:0"), torch.empty(2000, dtype=torch.float64, device="cuda:0")
        flags = torch.empty(2000, dtype=torch.uint8, device="cuda:0")
        B.rmpc_trace_debug(ctx, mid, x, 2000, P, hit.data_ptr(), d.data_ptr(), flags.data_ptr())
        return hit.cpu(), d.cpu()

    try:
        before = arena.clone()
        mid = upload()
        changed = torch.nonzero(arena != before).reshape(-1)
        base = int(changed[0]) // 256 * 256
        assert int(changed[-1]) >= base + own
        want = trace(mid)
        byte = torch.zeros(4096 * 4096, dtype=torch.uint8, device="cuda:0")
        for dims in ((4096, 1, 4096), (4096, 1, 512), (4096, 1, 64), (4096, 1, 8), (4096, 1, 1), (256, 1, 1)):
            while True:
                try:
                    B.rmpc_map_upload(ctx, *dims, "u8", 0.1, (0, 0, 0), byte.data_ptr(), True)
                except B.RmpcError as e:
                    assert e.status == B.RMPC_E_NOMEM
                    break
        B.rmpc_map_release(ctx, mid)
        got = trace(upload())
        assert all(torch.equal(a, b) for a, b in zip(want, got))
    finally:
        B.rmpc_destroy(ctx)


@pytest.mark.parametrize("enc,subvoxel", [("f32", 0), ("f32", 1), ("f16", 1), ("u8", 0)])
@pytest.mark.parametrize("at", [(8100, 8150, 20), (-8180, -8100, -8150)])
def test_far_queries_on_indexed_maps(ctx, tiny_map, enc, subvoxel, at):
    """Beyond 2^16 voxels from the origin a map's index serves as well as its table does (an upload
    without scratch has no index): bit for bit from starts among the blocks, beside them and out of
    reach of them, far from the origin and at the end of the allowed range."""
    sm = W.sparse_from_dense(tiny_map, offset_blocks=at, keep_free=0.3, seed=4, origin_m=(0.0, 0.0, 0.0))
    data = {"f32": sm.values, "f16": W.encode_f16(sm.values), "u8": W.encode_u8(sm.values)}[enc]
    far = ctx.upload_sparse(sm.coords, data, sm.voxel_m, sm.origin_m, enc)
    _limit(ctx, 0)
    mid = ctx.upload_sparse(sm.coords, data, sm.voxel_m, sm.origin_m, enc)
    lo = np.asarray(at) * 8.0
    p = dict(P, max_range=40.0, subvoxel=subvoxel)                      # 400 voxels
    starts = [lo + g for g in ((17.3, 40.6, 30.2), (50.01, 9.99, 33.5), (-300.4, 20.1, 30.7), (70.2, 90.3, -80.1), (32.0, 32.0, 70.0))]
    starts += [lo + 30000.7, np.full(3, 8.38e6), -np.full(3, 8.38e6)]
    hits = 0
    for g in starts:
        x = sm.origin_m + g * sm.voxel_m
        a, b = ctx.trace(far, x, 4096, p), ctx.trace(mid, x, 4096, p)
        for k in ("hit", "d", "visits"):
            assert np.array_equal(a[k], b[k]), (g, k)
        assert np.array_equal(a["flags"] & 0xfe, b["flags"] & 0xfe), g
        hits += int((a["hit"] >= 0).sum())
        v = np.array([1.0, -0.5, 0.3])
        _same_query(ctx.query(far, x, v, 3000, p), ctx.query(mid, x, v, 3000, p))
        if not subvoxel:
            q = [dict(kind="map", map_id=m, n=700, x=x, v=v) for m in (far, mid)]
            _same_query(*ctx.query_batch(q, p, None))
    assert hits > 4096
