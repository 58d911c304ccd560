"""Point location and NavSafety through the daughter indexes (radial order, phi
sectors, padded boxes), against the oracle's loop over every daughter.

The points sit where an index can go wrong: on the axis and within 1e-7 mm of
it, on every tube's radii and between neighbouring tubes, on sector borders, on
daughters' faces and just off them, beyond the mothers' ends, far outside the
world and at infinity, and uniform in the world.  Points within the oracle's
band-edge margin of a surface may be told apart by rounding alone: they are the
ones whose nearest signed term is within 1e-11 of the band's edge, and none of
the constructed offsets (0, 1e-10, 1e-8, 1e-3 mm) is.

Bar: volumes exact; safeties within 1e-12 max(|ref|, 1 mm)."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import compare_values, cuda, host, say

pytestmark = pytest.mark.gpu


def steep_description():
    """Flat cones and a Trd with slopes of 100 to 2000, mixed types: the boxes
    index, with a surface band that reaches far along the axes."""
    lvs = [W.LV(W.box(300.0, 300.0, 100.0), [])]
    for k, s in enumerate([W.cons(0.0, 5.0, 0.0, 45.0, 0.2), W.cons(3.0, 40.0, 0.0, 4.0, 0.01),
                           W.trd(1.0, 41.0, 40.0, 2.0, 0.01), W.sphere(5.0, 30.0),
                           W.pcon([-1.0, 0.0, 0.01, 5.0], [0.0, 0.0, 1.0, 0.0], [40.0, 5.0, 45.0, 45.0])]):
        R = W._rot((1.0, 2.0, k), 0.4 * k)
        lvs[0].placements.append((k + 1, R, np.array([-200.0 + 100.0 * k, 60.0 * (k % 3 - 1), 3.0 * k])))
        lvs.append(W.LV(s, []))
    return lvs


CASES = {
    "detector": (lambda: W.detector_description()[0], W.WORLD_HALF),
    "nested_tubes": (W.nested_tubes_description, (400.0, 400.0, 400.0)),
    "ring": (W.ring_description, (200.0, 200.0, 200.0)),
    "grid": (W.grid_description, (200.0, 200.0, 200.0)),
    "big_grid": (W.big_grid_description, (200.0, 200.0, 200.0)),
    "bundle": (W.bundle_description, (200.0, 200.0, 200.0)),
    "composites": (W.composite_description, (300.0, 300.0, 300.0)),
    "steep": (steep_description, (300.0, 300.0, 100.0)),
}


def special_points(lvs, half, rng):
    """Points on and near the surfaces of every placed volume (at most 40 of
    them), the axis, the sector borders and the far field."""
    out = []
    tree = W.expand_pvs(lvs)
    for lv, _, R, t, _ in [tree[i] for i in rng.choice(len(tree), min(40, len(tree)), replace=False)]:
        p, nrm = W.sample_surface(lvs[lv].solid, rng, 64)
        for e in (0.0, 1e-10, -1e-10, 1e-8, -1e-8, 1e-3, -1e-3):
            out.append((R @ (p + e * nrm)).T + t)
    z = rng.uniform(-half[2], half[2], 64)
    for r in (0.0, 1e-300, 1e-9, 1e-7, 2e-6, 1e-3):
        phi = rng.uniform(0.0, W.TWO_PI, 64)
        out.append(np.stack([r * np.cos(phi), r * np.sin(phi), z], 1))
    for s in range(256):  # the borders of the pseudo-angle sectors
        a = s / 64.0
        f = a - math.floor(a)
        u, v = (1.0 - f, f) if a < 1 else ((-f, 1.0 - f) if a < 2 else ((f - 1.0, -f) if a < 3 else (f, f - 1.0)))
        r = rng.uniform(1.0, half[0], 4)
        out.append(np.stack([r * u, r * v, rng.uniform(-20.0, 20.0, 4)], 1))
    out.append(rng.uniform(-1.0, 1.0, (64, 3)) * 1e9)
    far = rng.uniform(-10.0, 10.0, (6, 3))
    far[np.arange(6), np.arange(6) % 3] = np.where(np.arange(6) < 3, np.inf, -np.inf)
    out.append(far)
    out.append(rng.uniform(-1.02, 1.02, (20011, 3)) * np.asarray(half))
    return np.concatenate(out).T.copy()


@pytest.mark.parametrize("name", list(CASES))
def test_lookup(name):
    import paper_1512_06637_amd as G
    desc, half = CASES[name]
    lvs = desc()
    blob = W.make_blob(lvs)
    rng = np.random.default_rng(91)
    x, y, z = special_points(lvs, half, rng)
    og = O.Geometry(blob)
    ref = og.locate(x, y, z)
    with G.Geometry(blob) as g:
        a = [cuda(v) for v in (x, y, z)]
        got = host(g.locate(*a))
        assert np.array_equal(got, ref), (name, np.nonzero(got != ref)[0][:8])
        # safeties: in the located volume, and in its mother (points in or on a daughter)
        parent = np.array([p for _, p, _, _, _ in W.expand_pvs(lvs)], np.int32)
        for pv in (ref, np.where(ref > 0, parent[np.maximum(ref, 0)], ref).astype(np.int32)):
            keep = np.isfinite(x + y + z) & (pv >= 0)
            b = [np.ascontiguousarray(v[keep]) for v in (x, y, z)]
            p = np.ascontiguousarray(pv[keep].astype(np.int32))
            want = og.nav_safety(*b, p)
            for prec in (G.FP64, G.FP32_REFINE):
                s = host(g.nav_safety(*[cuda(v) for v in b], cuda(p), precision=prec))
                _, _, bad = compare_values(s, want, what=f"{name} safety")
                assert bad.size == 0, (name, prec, bad[:8])
    say(f"  {name}: {x.size} points, {int((ref >= 0).sum())} in the world, {len(set(ref.tolist()))} volumes")
