"""Point lookups among daughters found by masks of 64 padded boxes, at the edges
of the masks: a row of boxes that touch, placed in a shuffled order, so that a
point on a shared face belongs to the first of its two boxes, wherever in the
masks they lie.  Volumes are exact, against the oracle."""
import numpy as np
import pytest

import oracle as O
from paper_1512_06637_amd import workloads as W
from tests.gpu_util import cuda, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 63, 64, 65, 128, 129])
def test_touching_boxes(count):
    import paper_1512_06637_amd as G
    rng = np.random.default_rng(count)
    half = count + 1.0
    lvs = [W.LV(W.box(half, 3.0, 3.0), []), W.LV(W.box(1.0, 1.0, 1.0), [])]
    centre = 2.0 * np.arange(count) - (count - 1)
    for c in centre[rng.permutation(count)]:
        lvs[0].placements.append((1, np.eye(3), np.array([c, 0.0, 0.0])))
    blob = W.make_blob(lvs)
    faces = np.repeat(np.append(centre - 1.0, centre[-1] + 1.0), 8)
    x = np.concatenate([faces, rng.uniform(-half, half, 4099)])
    y, z = rng.uniform(-1.5, 1.5, (2, len(x)))
    mix = rng.permutation(len(x))
    x, y, z = (np.ascontiguousarray(v[mix]) for v in (x, y, z))
    ref = O.Geometry(blob).locate(x, y, z)
    with G.Geometry(blob) as g:
        got = host(g.locate(cuda(x), cuda(y), cuda(z)))
    assert np.array_equal(got, ref)
    assert len(np.unique(ref)) > count  # the world outside the row, and every box
