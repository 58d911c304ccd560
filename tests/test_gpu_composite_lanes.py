"""Composites beside other solids, against the oracle: a detector with one
composite (or one cone) in a kind of module or in the world, and many composites,
each a logical volume of its own, up to where the start groups of the transports'
order leave no bits for the direction, no group per daughter, and no groups.
Location, single steps, safeties and whole transports, where the lanes of a
wavefront sit in different composites and in the same one.

Bar: volumes, sequences, counts and flags exact for tracks the oracle does not
flag; single steps and safeties within 1e-12 max(|ref|, 1 mm).  The lengths along
a transport drift with the point advanced by both codes (128 steps up to 3.5 m from
the origin here, with no bound on the angle of a hit): the lengths of the two
forms equal each other bit for bit instead."""
import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import compare_values, cuda, host, transport_bits_equal

pytestmark = pytest.mark.gpu

E = np.eye(3)


def detector(solid, where):
    lvs, _ = W.detector_description()
    lvs.append(W.LV(solid, []))
    if where == "world":
        lvs[0].placements.append((len(lvs) - 1, E, np.array([0.0, 0.0, 2750.0])))
    else:  # the modules of layer 5
        lvs[12].placements.append((len(lvs) - 1, E, np.zeros(3)))
    return lvs


def cells(slabs, per_slab, kids=0):
    """A world of slabs, each holding per_slab composites (bored boxes), every one
    a logical volume of its own; kids: instead boxes of their own, each holding
    that many placements of one small composite."""
    lvs = [W.LV(W.box(700.0, 700.0, 700.0), [])]
    hz = 0.8 * 600.0 / slabs
    m = int(np.ceil(np.sqrt(per_slab)))
    h = 0.8 * 580.0 / m
    if kids:
        lvs.append(W.LV(W.boolean(W.SUBTRACTION, W.box(0.4 * h / 8, 0.8 * h, 0.5 * hz), W.tubs(0.0, 0.3 * h / 8, 900.0)), []))
    for i in range(slabs):
        slab = W.LV(W.box(600.0, 600.0, hz), [])
        lvs[0].placements.append((len(lvs), E, np.array([0.0, 0.0, -600.0 + 1200.0 * (i + 0.5) / slabs])))
        lvs.append(slab)
        for j in range(per_slab):
            at = np.array([580.0 * (2 * (j % m) + 1 - m) / m, 580.0 * (2 * (j // m) + 1 - m) / m, 0.0])
            slab.placements.append((len(lvs), E, at))
            if kids:
                lvs.append(W.LV(W.box(h, h, 0.9 * hz), [(1, E, np.array([h * (2 * k + 1 - kids) / kids, 0.0, 0.0]))
                                                         for k in range(kids)]))
            else:
                lvs.append(W.LV(W.boolean(W.SUBTRACTION, W.box(h, h, 0.6 * hz), W.tubs(0.0, 0.4 * h, 900.0)), []))
    return lvs


BORED = W.boolean(W.SUBTRACTION, W.box(12.0, 3.0, 100.0), W.tubs(0.0, 2.0, 200.0))
BLOCK = W.boolean(W.SUBTRACTION, W.box(200.0, 200.0, 100.0), W.tubs(0.0, 100.0, 200.0))
CASES = {
    "composite in modules": (lambda: detector(BORED, "modules"), W.WORLD_HALF, 8211),
    "composite in world": (lambda: detector(BLOCK, "world"), W.WORLD_HALF, 8211),
    "cone in modules": (lambda: detector(W.cons(2.0, 8.0, 1.0, 12.0, 100.0), "modules"), W.WORLD_HALF, 8211),
    "300 composites": (lambda: cells(6, 49), (650.0,) * 3, 8211),
    "700 composites": (lambda: cells(10, 70), (650.0,) * 3, 8211),
    "8300 composites": (lambda: cells(91, 91), (650.0,) * 3, 2049),  # no bits left for the direction
    "groups without bins": (lambda: cells(4, 140, 15), (650.0,) * 3, 8211),  # 561 x 31 groups would be too many
    "no groups": (lambda: cells(130, 127), (650.0,) * 3, 1025),  # more than 16,384 volumes
}


@pytest.mark.parametrize("name", list(CASES))
def test_navigation(name):
    import paper_1512_06637_amd as G
    make, half, n = CASES[name]
    lvs = make()
    blob = W.make_blob(lvs)
    t = W.uniform_world_tracks(half, n, 900 + n)
    t.x[:65] = np.linspace(-1.0, 1.0, 65)  # and starts near the origin
    t.y[:65] = t.z[:65] = 0.25
    og = O.Geometry(blob)
    start = og.locate(t.x, t.y, t.z).astype(np.int32)
    rst, rnx, rfl, rdg = og.step(t, start)
    rsf = og.nav_safety(t.x, t.y, t.z, start)
    rsf, sdg = rsf if isinstance(rsf, tuple) else (rsf, None)
    ref = og.transport(t)
    ok = (rdg & O.D_ILL) == 0
    with G.Geometry(blob) as g:
        a = [cuda(v) for v in t.arrays()]
        pv = g.locate(*a[:3])
        assert np.array_equal(host(pv), start)
        for prec in (G.FP64, G.FP32_REFINE):
            st, nx = g.step(*a, pv, precision=prec)
            assert np.array_equal(host(nx)[ok], rnx[ok])
            assert compare_values(host(st)[ok], rst[ok], what=f"{name}: step")[2].size == 0
            sf = host(g.nav_safety(*a[:3], pv, precision=prec))
            assert compare_values(sf, rsf, sdg, what=f"{name}: safety")[2].size == 0
        first = None
        for form in (0, 1):
            g.set_tuning(transport=form)
            for prec in (G.FP64, G.FP32_REFINE):
                for begin in (None, pv):
                    got = g.transport(*a, start_pv=begin, precision=prec)
                    if first is None:
                        first = got
                        good = (ref["diag"] & O.D_ILL) == 0
                        assert good.sum() > 0.9 * n
                        assert np.array_equal(host(got["nsteps"])[good], ref["nsteps"][good])
                        assert np.array_equal(host(got["flags"])[good], ref["flags"][good])
                        k = (np.arange(129)[None, :] <= ref["nsteps"][:, None]) & good[:, None]
                        assert np.array_equal(host(got["pv"])[k], ref["pv"][k])
                    else:
                        assert transport_bits_equal(got, first), (form, prec)
