"""DistanceToIn/Out of full tubes (the closed form without phi faces) against
the oracle: solid cylinders, thin and thick shells, and radii beyond the 1e5 mm
up to which the square root of the radius is skipped.

Rays from points on and near every surface (exactly on it, 1e-10, 3e-10, 1e-8,
1e-3 mm off, and one rounding off the radius), on the axis, and uniform around
the solid, moving radially, tangentially (B = 0), along the generator and the
axis (A = 0), through the axis, and isotropically.

Bar: 1e-12 max(|ref|, 1 mm), sentinels exact, on tracks the oracle does not
flag; a band point's Inside code decides the sentinel, so points within the
oracle's band-edge margin are flagged by it."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import compare_values, cuda, host

pytestmark = pytest.mark.gpu

TUBES = [(0.0, 12.0, 30.0), (5.0, 15.0, 20.0), (49.999, 50.0, 7.0), (1890.0, 1930.0, 2500.0), (0.0, 2e5, 1e3),
         (1.5e5, 1.6e5, 2e4), (1e-3, 2e-3, 1.0)]


def rays(rmin, rmax, dz, n, rng):
    k = n // 8
    r = rng.choice([rmin, rmax], 4 * k)
    off = rng.choice([0.0, 1e-10, -1e-10, 3e-10, -3e-10, 1e-8, -1e-8, 1e-3, -1e-3], 4 * k)
    r = np.abs(r + off)
    r[::5] = np.nextafter(r[::5], rng.choice([0.0, np.inf], r[::5].size))
    ph = rng.uniform(0, W.TWO_PI, 4 * k)
    ph[::3] = rng.choice([0.0, math.pi / 2, math.pi], ph[::3].size)
    z = rng.uniform(-1.2 * dz, 1.2 * dz, 4 * k)
    face = np.arange(4 * k) % 4 == 0
    z[face] = rng.choice([-dz, dz], int(face.sum())) + off[face]
    r[face] = rng.uniform(0.0, 1.3 * rmax, int(face.sum()))
    axis = np.zeros(k)
    P = np.concatenate([np.stack([r * np.cos(ph), r * np.sin(ph), z]),
                        np.stack([axis, axis, rng.uniform(-2 * dz, 2 * dz, k)]),
                        rng.uniform(-2.0, 2.0, (3, n - 5 * k)) * np.array([rmax, rmax, dz])[:, None]], axis=1)
    D = np.stack(W.isotropic(rng, n))
    rad = np.hypot(P[0], P[1])
    u = np.where(rad > 0, P[:2] / np.where(rad > 0, rad, 1.0), np.array([[1.0], [0.0]]))
    kind = rng.integers(0, 8, n)
    sg = rng.choice([-1.0, 1.0], n)
    zero = np.zeros(n)
    D = np.where(kind == 0, np.stack([sg * u[0], sg * u[1], zero]), D)
    D = np.where(kind == 1, np.stack([-sg * u[1], sg * u[0], zero]), D)
    D = np.where(kind == 2, np.stack([zero, zero, sg]), D)
    D = np.where(kind == 3, np.stack([-0.6 * u[0], -0.6 * u[1], 0.8 * sg]), D)
    return W.Tracks(*[np.ascontiguousarray(v) for v in np.concatenate([P, D])])


@pytest.mark.parametrize("tube", TUBES)
def test_full_tube(tube):
    import paper_1512_06637_amd as G
    s = W.tubs(*tube)
    t = rays(*tube, 20000, np.random.default_rng(17))
    with G.Geometry(W.single_solid_blob(s)) as g:
        a = [cuda(v) for v in t.arrays()]
        for d in (G.TO_IN, G.TO_OUT):
            ref, diag = O.distance(s, d, t)
            n_ok, _, bad = compare_values(host(g.distance(0, d, *a)), ref, diag, what=f"full tube {tube} {d}")
            assert bad.size == 0, (tube, d, bad[:5])
            assert ((diag & O.D_ILL) == 0).sum() > 0.4 * t.n
