"""Policy parameters at the ends of float32: rays whose terms are all zero may be left out of the sums,
but only where every term is zero; a term that is not a number stays one.  The sums against the same
float32 formulas evaluated for every ray."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2301_08068_amd import workloads as W  # noqa: E402

F = np.float32
BASE = W.params("static", max_range=5.0)
# beyond float32 both ways, and either side of where the kernels stop leaving rays out
EXTREMES = [dict(), dict(c=1e-31), dict(c=1e-29), dict(c=1e-46), dict(c=0.9e38), dict(c=2e38), dict(c=1e39), dict(eta_rep=0.9e30),
            dict(eta_rep=1.1e30), dict(eta_rep=1e39), dict(nu_rep=1e-38), dict(nu_rep=1e-40), dict(nu_rep=1e50), dict(radius=1e-38),
            dict(radius=1e-40), dict(radius=1e-50), dict(radius=1e50), dict(nu_damp=1e-40), dict(eps=1e-50), dict(eta_damp=1e39),
            dict(eta_damp=0.0), dict(nu_rep=1e-40, radius=1e-40)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_08068_amd import binding
    c = binding.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


def _sums(p, v, r, d):
    """The 9 sums of all rays' terms (S upper triangle, b) in float64, nan where a term is not finite."""
    with np.errstate(all="ignore"):
        c, eta_rep, eta_damp, radius, eps = (F(p[k]) for k in ("c", "eta_rep", "eta_damp", "radius", "eps"))
        inv_rep, inv_damp, inv_rad = (F(1.0 / np.float64(p[k])) for k in ("nu_rep", "nu_damp", "radius"))
        v = v.astype(F)
        vr = v[0] * r[:, 0] + v[1] * r[:, 1] + v[2] * r[:, 2]
        pp = np.where(vr > 0, vr * vr, F(0))
        q = eta_damp * pp / (d * inv_damp + eps)
        rn2 = (r * r).sum(axis=1, dtype=F)
        mq = q * np.sqrt(rn2)
        sigma = q / (mq + c * np.log1p(np.exp(F(-2) * c * mq)))
        wl = F(1) - d * inv_rad
        a = np.where(d <= radius, wl * wl, F(0)) * sigma * sigma
        phi = eta_rep * np.exp(-d * inv_rep) + q
        bb = -a * rn2 * phi
        t = [a * r[:, i] * r[:, j] for i in range(3) for j in range(i, 3)] + [bb * r[:, i] for i in range(3)]
        t = np.stack(t).astype(np.float64)
        return np.where(np.isfinite(t).all(axis=1), t.sum(axis=1), np.nan)


def _check(g, want):
    got = np.concatenate([g["S"][np.triu_indices(3)], g["b"]])
    assert np.array_equal(np.isnan(got), np.isnan(want)), (got, want)
    for part in (slice(0, 6), slice(6, 9)):
        scale = np.nanmax(np.abs(want[part]), initial=0.0)
        # 1e-4 of the largest sum, as for every float32 policy against its reference
        assert np.all(np.isnan(want[part]) | (np.abs(got[part] - want[part]) <= 1e-4 * scale)), (got, want)


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("extreme", EXTREMES, ids=str)
def test_scan_terms(ctx, extreme, far):
    """Points all round at 0.3 to 4 m, or one at 1e38 m along each axis besides (whose float32 distance
    overflows), with the robot moving away from half of them."""
    p = dict(BASE, min_range=0.0, **extreme)
    rng = np.random.default_rng(3)
    pts = rng.normal(size=(500, 3))
    pts = (pts / np.linalg.norm(pts, axis=1, keepdims=True) * rng.uniform(0.3, 4.0, (500, 1))).astype(F)
    if far:
        pts = np.concatenate([pts, np.full((1, 3), 3e38, F)])
    v = np.array([-1.0, -0.5, -0.3])
    d64 = np.sqrt((pts.astype(np.float64) ** 2).sum(axis=1))
    with np.errstate(over="ignore"):
        want = _sums(p, v, pts * (1.0 / d64).astype(F)[:, None], d64.astype(F))
    _check(ctx.scan_query(pts, v, p), want)


@pytest.mark.parametrize("extreme", EXTREMES, ids=str)
def test_map_terms_at_distance_zero(ctx, extreme):
    """A start in an occupied voxel: every ray hits at distance 0."""
    p = dict(BASE, **extreme)
    mid = ctx.upload(np.full((4, 4, 4), -0.1, F), 0.5, np.zeros(3), "f32")
    try:
        r = ctx.directions(1000)
        v = np.array([1.0, 0.2, -0.4])
        _check(ctx.query(mid, [1.1, 0.9, 1.2], v, 1000, p), _sums(p, v, r, np.zeros(1000, F)))
    finally:
        ctx.release(mid)
