"""Polycone queries against the oracle where the section walk and its kernels
can go wrong: the fewest and the most planes (2, 64), radii that step, taper and
reach zero, inner cones on some sections only, rays that pass sections outside
their radius, horizontal and vertical rays, baskets at the edges of a wavefront
and of a workgroup, and DistanceToOut on both sides of the basket size from
which its walks are compacted (the rays of a small basket, repeated).

Bar: 1e-12 max(|ref|, 1 mm), sentinels exact, on tracks the oracle does not flag."""
import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import compare_values, cuda, host

pytestmark = pytest.mark.gpu


def polycone(kind):
    if kind == "two planes":
        return W.pcon([-7.0, 9.0], [0.0, 1.0], [5.0, 11.0])
    if kind == "hollow in part":
        return W.pcon([-30.0, -10.0, -9.5, 12.0, 40.0], [0.0, 0.0, 4.0, 4.0, 0.0], [20.0, 8.0, 30.0, 30.0, 0.5])
    k = np.arange(64)
    z = np.cumsum(np.where(k % 2 == 0, 0.5, 6.0)) - 100.0
    rmax = np.where(k % 4 < 2, 25.0, 60.0) + 0.1 * k
    return W.pcon(z, np.where(k > 40, 5.0, 0.0), rmax)


def rays(s, n, rng):
    c, h = W.solid_extent(s)
    P = np.asarray(c)[:, None] + rng.uniform(-1.6, 1.6, (3, n)) * np.asarray(h)[:, None]
    P[:, ::3] *= 0.5  # more of them inside
    D = np.stack(W.isotropic(rng, n))
    D[:, 1::8] = np.array([0.0, 0.0, 1.0])[:, None] * rng.choice([-1.0, 1.0], n)[1::8]
    D[2, 2::8] = 0.0
    D[:, 2::8] /= np.linalg.norm(D[:, 2::8], axis=0)
    return W.Tracks(*[np.ascontiguousarray(v) for v in np.concatenate([P, D])])


@pytest.mark.parametrize("n", [1, 63, 65, 257, 20000])
@pytest.mark.parametrize("kind", ["two planes", "hollow in part", "64 planes"])
def test_polycone(kind, n):
    import torch

    import paper_1512_06637_amd as G
    s = polycone(kind)
    t = rays(s, n, np.random.default_rng(31))
    with G.Geometry(W.single_solid_blob(s)) as g:
        a = [cuda(v) for v in t.arrays()]
        code = torch.empty(n, dtype=torch.int8, device="cuda")
        out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(3)]
        g.solid_all(0, *a, code, *out)
        single = {"safety": g.safety(0, *a[:3])}
        for d in (G.TO_IN, G.TO_OUT):
            single[d] = g.distance(0, d, *a)
            ref, diag = O.distance(s, d, t)
            for got in (single[d], out[1 + d]):
                _, _, bad = compare_values(host(got), ref, diag, what=f"polycone {kind} {n} {d}")
                assert bad.size == 0, (kind, n, d, bad[:5])
            assert n < 100 or ((diag & O.D_ILL) == 0).mean() > 0.9
        assert torch.equal(code, g.inside(0, *a[:3]))
        assert torch.allclose(out[0], single["safety"], rtol=1e-12, atol=1e-12)
        if n == 20000:
            m = (1 << 19) + 65
            many = [v.repeat(m // n + 1)[:m].contiguous() for v in a]
            ref, diag = O.distance(s, G.TO_OUT, t)
            for k in (m, (1 << 19) - 1):
                got = host(g.distance(0, G.TO_OUT, *[v[:k].contiguous() for v in many]))
                r = np.arange(k) % n
                _, _, bad = compare_values(got, ref[r], diag[r], what=f"polycone {kind} {k} out")
                assert bad.size == 0, (kind, k, bad[:5])
