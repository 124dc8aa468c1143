"""The RANSAC kernel decides most inlier tests from a float32 form of
d^2 - mid with an error bound E, and leaves those with |e| <= E to the float64
test.  This repeats the form on the CPU (float32 coefficients, a chain of fused
multiply-adds from z on, as the matrix unit evaluates it) and checks that every
decided test is the float64 one: random triples' circles, circles with lattice
points a hair from either edge of the band, nearly straight lines, bands wider
than the radius, at frame sizes from 16 x 16 to 16384 x 16384."""
import numpy as np
import pytest

f32, f64 = np.float32, np.float64


def fma32(a, b, c):
    # a b is exact in float64; the sum is rounded to 53 bits, then to 24: it
    # can differ from one rounding only at a tie of the second, by 2^-29 ulp
    return (a.astype(f64) * b.astype(f64) + c.astype(f64)).astype(f32)


def band(r2, t):
    r = np.sqrt(r2)
    return np.where(r > t, (r - t) ** 2, -1.0), (r + t) ** 2


def quick(cx, cy, lo2, hi2, U, V):
    mid, half = 0.5 * (lo2 + hi2), (0.5 * (hi2 - lo2)).astype(f32)
    x, y = (-2.0 * cx).astype(f32), (-2.0 * cy).astype(f32)
    k = ((cx * cx + cy * cy) - mid).astype(f32)
    U, V = f32(U), f32(V)
    S = ((U * U + V * V) + np.abs(x) * U + np.abs(y) * V + np.abs(k)).astype(f32)
    E = (f32(2.0 ** -22) * S + f32(2.0 ** -21) * half).astype(f32)
    m = min(U, V)
    return x, y, k, half, E, S < f32(2.0 ** 26) * m * m


def decided_share(cx, cy, r2, t, u, v, U, V):
    """Asserts every decided test; returns the share that is decided."""
    lo2, hi2 = band(r2, t)
    x, y, k, half, E, on = quick(cx, cy, lo2, hi2, U, V)
    uf, vf = u.astype(f32)[None, :], v.astype(f32)[None, :]
    z = ((u * u + v * v).astype(f32))[None, :]
    one = np.ones_like(z)
    d = fma32(one, k[:, None], fma32(vf, y[:, None], fma32(uf, x[:, None], z)))
    e = (np.abs(d) - half[:, None]).astype(f32)
    sure = (np.abs(e) > E[:, None]) & on[:, None]
    du, dv = u.astype(f64)[None, :] - cx[:, None], v.astype(f64)[None, :] - cy[:, None]
    d2 = du * du + dv * dv
    exact = (lo2[:, None] <= d2) & (d2 <= hi2[:, None])
    assert np.array_equal((e < 0)[sure], exact[sure])
    return float(sure.mean())


def triple_circles(u, v, rng, n):
    i = rng.integers(0, len(u), (n, 3))
    x, y = u[i].astype(object), v[i].astype(object)
    out = []
    for (x0, x1, x2), (y0, y1, y2) in zip(x, y):
        D = 2 * (x0 * (y1 - y2) + x1 * (y2 - y0) + x2 * (y0 - y1))
        if D == 0:
            continue
        z0, z1, z2 = x0 * x0 + y0 * y0, x1 * x1 + y1 * y1, x2 * x2 + y2 * y2
        cx = float(z0 * (y1 - y2) + z1 * (y2 - y0) + z2 * (y0 - y1)) / float(D)
        cy = float(z0 * (x2 - x1) + z1 * (x0 - x2) + z2 * (x1 - x0)) / float(D)
        out.append((cx, cy, (float(x0) - cx) ** 2 + (float(y0) - cy) ** 2))
    return [np.array(c, dtype=f64) for c in zip(*out)]


@pytest.mark.parametrize("W,H", [(16, 16), (640, 480), (1920, 1080), (3840, 2160), (512, 16384),
                                 (16384, 16384)])
def test_decided_tests_are_the_float64_ones(W, H):
    rng = np.random.default_rng(W + H)
    ox, oy = W // 2, H // 2
    U, V = max(ox, W - 1 - ox), max(oy, H - 1 - oy)
    u, v = rng.integers(0, W, 200) - ox, rng.integers(0, H, 200) - oy
    shares = []
    for t in (0.0, 0.5, 3.0, 40.0):
        shares.append(decided_share(*triple_circles(u, v, rng, 2000), t, u, v, U, V))
        # points of two neighbouring columns or rows: nearly straight lines
        a = np.concatenate([rng.integers(0, 3, 100) - ox, rng.integers(0, W, 100) - ox])
        b = np.concatenate([rng.integers(0, H, 100) - oy, rng.integers(0, 3, 100) - oy])
        decided_share(*triple_circles(a, b, rng, 2000), t, a, b, U, V)
        # a lattice point a few units in the last place from a band edge
        cx, cy = rng.uniform(-U, U, 500), rng.uniform(-V, V, 500)
        dist = np.hypot(u[:500 % 200 or 200][0] - cx, v[0] - cy)
        for sign in (-1.0, 1.0):
            for ulps in (-4, 0, 4):
                r = np.abs(dist + sign * t)
                r2 = (r * (1.0 + ulps * 2.0 ** -52)) ** 2
                decided_share(cx, cy, r2, t, u, v, U, V)
    assert max(shares) > 0.99    # the float32 form is worth taking
