"""Point lookups around 256 points per CU, below which the chip is not full and a
daughter's tables are waited for, against the oracle: 25 boxes, 12 tilted tubes,
boxes in composites."""
import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import cuda, host

pytestmark = pytest.mark.gpu

GEO = {"grid": (W.grid_description, 130.0), "bundle": (W.bundle_description, 130.0), "composites": (W.composite_description, 290.0)}


@pytest.mark.parametrize("extra", [-1, 0, 1, 64])
@pytest.mark.parametrize("name", list(GEO))
def test_locate_at_the_switch(name, extra):
    import torch
    import paper_1512_06637_amd as G
    make, half = GEO[name]
    blob = W.make_blob(make())
    n = 256 * torch.cuda.get_device_properties(0).multi_processor_count + extra
    t = W.uniform_world_tracks((half,) * 3, n, 31 + extra)
    t.x[::9], t.y[::9] = np.round(t.x[::9]), np.round(t.y[::9])  # points on faces of boxes among them
    ref = O.Geometry(blob).locate(t.x, t.y, t.z)
    with G.Geometry(blob) as g:
        got = host(g.locate(cuda(t.x), cuda(t.y), cuda(t.z)))
    assert np.array_equal(got, ref)
    assert len(np.unique(ref)) > 5
