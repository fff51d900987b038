"""The implicit surface: intersections, launches and leaf cells depend on the leaf size alone, not on the levels above
it: also with levels that divide nothing (ratio 1) and with the smallest ratios, where a sample's 27 leaves lie in
several bricks."""
import numpy as np
import pytest

import scenes
from tests.test_gpu_sdf_routes import _rays, _same
from tests.test_gpu_walk import _stretched

pytestmark = pytest.mark.gpu


def _scene(pcrl, s, levels, compact=False):
    return pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), compact=compact)


@pytest.mark.parametrize("compact", [False, True])
@pytest.mark.parametrize("extent,levels", [
    (6.0, (0.2, 0.2)), (6.0, (0.2, 0.2, 0.2)), (6.0, (0.2, 0.2, 0.2, 0.2)), (6.0, (0.4, 0.2)), (6.0, (0.4, 0.2, 0.2)),
    (6.0, (0.6, 0.2, 0.2)), (6.0, (0.4, 0.4, 0.2)), (6.0, (0.8, 0.4, 0.2)), (6.0, (1.0, 1.0, 0.2, 0.2)),
    (6.0, (0.8, 0.2, 0.2, 0.2)),
    # the parents' grid would hold 9 G cells: after the equal levels, the top grid holds the parents again, or not
    (420.0, (3.2, 0.2, 0.2)), (420.0, (32.0, 1.6, 0.2, 0.2)), (420.0, (32.0, 0.8, 0.2, 0.2)),
])
def test_intersections_depend_on_the_leaf_size_alone(extent, levels, compact):
    import torch
    import paper_2402_13747_amd as pcrl
    s = _stretched(extent)
    flat = (3.2, 0.2) if extent > 100 else (0.2,)
    o, d = _rays(torch, s, 6000)
    ref, got = (pcrl.sdf_intersect(_scene(pcrl, s, l, compact), o, d) for l in (flat, levels))
    assert int((ref["leaf_cell"][:, 0] >= 0).sum()) > 1000
    _same(ref, got)


@pytest.mark.parametrize("levels", [(0.25, 0.25), (0.5, 0.25, 0.25), (0.25, 0.25, 0.25, 0.25)])
def test_launches_depend_on_the_leaf_size_alone(levels):
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    logs = []
    for l in ((0.25,), levels):
        L = pcrl.launch_rays(_scene(pcrl, s, l), s.tx, s.rx, n_rays=9000, max_reflections=3, hit_log=True, sdf=True)
        logs.append([x.cpu().numpy() for x in L.hit_log])
    assert (logs[0][0] >= 0).sum() > 9000  # a closed room: most rays go on
    for a, b in zip(*logs):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
