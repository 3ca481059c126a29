"""EDM on point sets whose squares leave the ordinary range: below 2^-100 (the
scaled root) down to the smallest subnormals, overflow, infinities, NaN,
coincident points, and mixtures that put all of them into one lane's four
elements.  Bit for bit against the correctly rounded root of the float32 sum
of squares fma(dz, dz, fma(dx, dx, dy dy)); both routes, both maps."""
import numpy as np
import pytest

import simplex_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def smap():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2208_11617_amd import binding
    binding.lib()
    return binding


def fma32(a, b, c):
    """a b + c of float32 arrays, rounded once: the exact product and its sum with
    c in float64, rounded to odd, then to float32."""
    x, y = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = x + y
    t = s - x
    err = (x - (s - t)) + (y - t)
    odd = np.isfinite(s) & (err != 0) & ((s.view(np.int64) & 1) == 0)
    s = np.where(odd, np.nextafter(s, np.where(err > 0, np.inf, -np.inf)), s)
    return s.astype(np.float32)


def reference(pts, n):
    """The (n+1) x (n+1) distances (row x_2, column x_1) of points x_1 and n - x_2."""
    with np.errstate(all="ignore"):
        d = pts[None, :, :] - pts[::-1][:, None, :]
        dx, dy, dz = (np.ascontiguousarray(d[..., k]) for k in range(3))
        return np.sqrt(fma32(dz, dz, fma32(dx, dx, dy * dy)))


def clouds(n):
    rng = np.random.default_rng(40 + n)
    base = rng.uniform(-1, 1, (n + 1, 3)).astype(np.float32)
    for e in (-40, -48, -50, -51, -60, -70, -74, 60, 63, 64, 100):
        with np.errstate(over="ignore"):
            yield f"2^{e}", np.ldexp(base, e).astype(np.float32)
    # scales change from point to point: squares on both sides of 2^-100 in a lane
    yield "mixed", np.ldexp(base, rng.integers(-76, -44, (n + 1, 1))).astype(np.float32)
    yield "all scales", np.ldexp(base, rng.integers(-76, 66, (n + 1, 3))).astype(np.float32)
    some = np.repeat(base[: n // 4 + 1], 4, axis=0)[: n + 1]
    yield "coincident", np.ascontiguousarray(rng.permutation(some))
    odd = base.copy()
    odd[rng.integers(0, n + 1, 3), rng.integers(0, 3, 3)] = np.inf
    odd[rng.integers(0, n + 1, 2), rng.integers(0, 3, 2)] = -np.inf
    odd[rng.integers(0, n + 1, 2), rng.integers(0, 3, 2)] = np.nan
    odd[rng.integers(0, n + 1, 4)] = -0.0
    yield "infinite and NaN", odd


# rows that start at lines (63, 127: row parts with 64- and 128-cell tiles), and not
@pytest.mark.parametrize("n", [40, 63, 100, 127])
def test_edm_values(smap, n):
    inside = np.arange(n + 1)[None, :] + np.arange(n + 1)[:, None] <= n
    try:
        for name, pts in clouds(n):
            want = reference(pts, n)
            d_pts = torch.from_numpy(pts).cuda()
            for rho in (16, 32, 64, 128):
                smap.set_tile(2, "edm", rho)
                for launch in (smap.map_launch, smap.bb_launch):
                    print(f"edm n={n} {name} rho={rho} {launch.__name__}", flush=True)
                    out = torch.from_numpy(si.sentinel_box(2, n, np.uint32).view(np.int32)).cuda()
                    launch(2, n, "edm", d_pts, out)
                    torch.cuda.synchronize()
                    got = out.cpu().numpy().view(np.float32).reshape(n + 1, n + 1)
                    assert np.array_equal(got[inside], want[inside], equal_nan=True)
                    assert (got.view(np.uint32)[~inside] == si.SENTINEL_U32).all()
    finally:
        smap.set_tile(2, "edm", 0)
