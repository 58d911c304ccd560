"""Daughters of mixed types, culled by their padded boxes, and transports that
start in several volumes (ordered by start volume and the daughters on the
track's way), against the oracle: single steps and whole transports, lane and
basket forms, FP64 and FP32 screens, starts located and given, at sizes around
a wavefront and a workgroup.

Bar: the navigation bar (sequences, counts and flags exact for tracks the
oracle does not flag; steps within 1e-12 relative + 1e-10 mm); the forms equal
each other bit for bit.  On solids with slopes of up to 2000, where the drift of
a point moves a step by far more, the culled loop is instead held to the plain
loop's outputs bit for bit (which runs where a placement is no rotation: a
further daughter, far from everything, has an R scaled by 1 + 1e-6)."""
import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import compare_values, cuda, host, transport_bits_equal
from tests.test_gpu_lookup import steep_description
from tests.test_gpu_nav import compare_transport

pytestmark = pytest.mark.gpu

def tracks(half, n):
    t = W.uniform_world_tracks(half, n, 4000 + n)
    k = n // 8  # starts around a placed volume, and rays along the axes
    t.x[:k], t.y[:k], t.z[:k] = t.x[:k] * 0.1 - 170.0, t.y[:k] * 0.2, t.z[:k] * 0.2
    return t


@pytest.mark.parametrize("n", [1, 63, 65, 257, 4099, 20011])
def test_mixed_daughters(n):
    import paper_1512_06637_amd as G
    blob = W.composite_blob()
    t = tracks((300.0, 300.0, 300.0), n)
    og = O.Geometry(blob)
    ref = og.transport(t)
    start = og.locate(t.x, t.y, t.z).astype(np.int32)
    inside = start >= 0
    tt = t.take(np.nonzero(inside)[0])
    rst, rnx, _, rdg = og.step(tt, start[inside])
    ok = (rdg & O.D_ILL) == 0
    with G.Geometry(blob) as g:
        a = [cuda(v) for v in t.arrays()]
        first = None
        for form in (2, 1):
            g.set_tuning(transport=form)
            for prec in (G.FP64, G.FP32_REFINE):
                for pv in (None, cuda(start)):
                    got = g.transport(*a, start_pv=pv, precision=prec)
                    if first is None:
                        first = got
                        assert compare_transport(got, ref) >= 0.9 * n - 1
                    else:
                        assert transport_bits_equal(got, first), (form, prec)
        b = [cuda(v) for v in tt.arrays()]
        for prec in (G.FP64, G.FP32_REFINE):
            st, nx = g.step(*b, cuda(start[inside]), precision=prec)
            assert np.array_equal(host(nx)[ok], rnx[ok])
            _, _, bad = compare_values(host(st)[ok], rst[ok], what="composite step")
            assert bad.size == 0


@pytest.mark.parametrize("n", [65, 20011])
def test_steep_culled_equals_plain(n):
    import torch
    import paper_1512_06637_amd as G
    lvs = steep_description()
    t = tracks((300.0, 300.0, 100.0), n)
    a = [cuda(v) for v in t.arrays()]
    got = []
    for plain in (False, True):
        if plain:
            lvs[0].placements.append((4, 1.000001 * np.eye(3), np.array([250.0, 250.0, 60.0])))
            keep = ~((np.abs(t.x - 250) < 40) & (np.abs(t.y - 250) < 40) & (np.abs(t.z - 60) < 40))
        with G.Geometry(W.make_blob(lvs)) as g:
            pv = g.locate(*a[:3])
            st, nx = g.step(*a, pv)
            got.append((pv, st, nx, g.transport(*a)))
    (p0, s0, n0, r0), (p1, s1, n1, r1) = got
    # tracks that never meet the further daughter (placed volume 6)
    free = torch.tensor(keep, device="cuda") & (r1["pv"] != 6).all(1)
    assert int(free.sum()) > 0.9 * n
    for u, v in ((p0, p1), (s0, s1), (n0, n1)):
        assert torch.equal(u[free], v[free])
    assert transport_bits_equal({k: v[free] for k, v in r0.items()}, {k: v[free] for k, v in r1.items()})


def test_start_volumes_out_of_range():
    """Given start volumes outside [0, n_pv), mixed with good ones."""
    import paper_1512_06637_amd as G
    blob = W.composite_blob()
    t = tracks((300.0, 300.0, 300.0), 999)
    pv = O.Geometry(blob).locate(t.x, t.y, t.z).astype(np.int32)
    pv[::7], pv[1::7], pv[2::7] = -1, -5, 1 << 20
    with G.Geometry(blob) as g:
        r = g.transport(*[cuda(v) for v in t.arrays()], start_pv=cuda(pv))
        ns, fl, p0 = host(r["nsteps"]), host(r["flags"]), host(r["pv"])[:, 0]
    good = (pv >= 0) & (pv < 10)
    assert np.array_equal(p0, np.where(good, pv, -1)) and (ns[~good] == 0).all() and (ns[good] > 0).all()
    assert np.array_equal(fl[~good], np.where(pv[~good] == -1, 0, 4))


def test_shared_placements():
    """Volumes whose placement ranges overlap in the blob (the same range, and
    a part of it) against the same geometry with ranges of their own."""
    import struct
    import torch
    import paper_1512_06637_amd as G
    e = np.eye(3)
    kids = [(4, W.rot_z(0.4 * k), np.array([25.0 * (k - 1.5), 10.0 * (k % 2) - 5.0, 0.0])) for k in range(4)]
    lvs = [W.LV(W.box(300.0, 60.0, 60.0), [(1, e, [-180.0, 0.0, 0.0]), (2, e, [0.0, 0.0, 0.0]), (3, e, [180.0, 0.0, 0.0])]),
           W.LV(W.box(60.0, 40.0, 40.0), kids), W.LV(W.tubs(0.0, 59.0, 40.0), kids), W.LV(W.box(60.0, 40.0, 40.0), kids[1:]),
           W.LV(W.box(5.0, 4.0, 20.0), [(5, e, [0.0, 0.0, 1.0])]), W.LV(W.tubs(1.0, 3.0, 10.0), [])]
    own = W.make_blob(lvs)
    shared = bytearray(own)
    for lv, (off, cnt) in ((1, (3, 4)), (2, (3, 4)), (3, (4, 3))):
        struct.pack_into("<2i", shared, 32 + 32 * lv + 12, off, cnt)
    t = W.uniform_world_tracks((300.0, 60.0, 60.0), 9001, 5)
    a = [cuda(v) for v in t.arrays()]
    got = []
    for blob in (own, bytes(shared)):
        with G.Geometry(blob) as g:
            pv = g.locate(*a[:3])
            got.append((g.n_pv, pv, g.transport(*a), g.nav_safety(*a[:3], pv)))
    assert got[0][0] == got[1][0] and torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][3], got[1][3])
    assert transport_bits_equal(got[0][2], got[1][2])
    assert (host(got[0][1]) > 8).sum() > 100
