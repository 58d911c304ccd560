"""basket_step around the sizes from which its tracks are regrouped by volume
(128 tracks per CU for boxes and full tubes, 256 for other elementary solids,
never with composites), and around a tile of the first regrouped sizes, against
the oracle: volumes out of range among good ones.

Bar: the navigation bar (next volumes and flags exact for tracks the oracle does
not flag, steps within 1e-12 max(|ref|, 1 mm))."""
import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import compare_values, cuda, host
from tests.test_gpu_composite_lanes import detector

pytestmark = pytest.mark.gpu

GEO = {"tubes": (lambda: W.detector_description()[0], 128), "cone": (lambda: detector(W.cons(2.0, 8.0, 1.0, 12.0, 100.0), "modules"), 256),
       "composites": (W.composite_description, 128)}


@pytest.mark.parametrize("extra", [-1, 0, 1, 63, 255, 256, 257])
@pytest.mark.parametrize("name", list(GEO))
def test_step_at_the_switch(name, extra):
    import torch
    import paper_1512_06637_amd as G
    make, per_cu = GEO[name]
    lvs = make()
    blob = W.make_blob(lvs)
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + extra
    t = W.uniform_world_tracks((300.0,) * 3 if name == "composites" else W.WORLD_HALF, n, 70 + extra)
    rng = np.random.default_rng(n)
    og = O.Geometry(blob)
    pv = og.locate(t.x, t.y, t.z).astype(np.int32)
    ps = np.where(rng.random(n) < 0.3, rng.uniform(0.0, 100.0, n), np.inf)
    bad = rng.random(n) < 0.05
    pv[bad] = rng.choice([-1, -7, 1 << 29], int(bad.sum()))
    good = np.nonzero(~bad)[0]
    rst, rnx, rfl, rdg = og.step(t.take(good), pv[good], ps[good])
    ok = (rdg & O.D_ILL) == 0
    with G.Geometry(blob) as g:
        a = [cuda(v) for v in t.arrays()]
        for prec in (G.FP64, G.FP32_REFINE):
            fl = cuda(np.full(n, -3, np.int32))
            st, nx = g.step(*a, cuda(pv), cuda(ps), out_flags=fl, precision=prec)
            st, nx, fl = host(st), host(nx), host(fl).astype(np.uint32)
            assert (st[bad] == 0).all() and (nx[bad] == -1).all() and (fl[bad] == 4).all()
            assert np.array_equal(nx[good][ok], rnx[ok]) and np.array_equal(fl[good][ok], rfl[ok])
            assert compare_values(st[good][ok], rst[ok], what=f"{name} step")[2].size == 0
