"""Few rays over the implicit surface: each meets what it meets in a larger bundle (a wave hands a few leaves out at first
in calls of up to 8 rays, all of a bundle's rays go to waves up to 4,096)."""
import numpy as np
import pytest

from tests.test_gpu_sdf_routes import _rays, _same
from tests.test_gpu_walk import _stretched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extent,levels", [(6.0, (0.3,)), (6.0, (1.0, 0.2)), (6.0, (0.2, 0.2)), (6.0, (2.0, 1.0, 0.2)),
                                           (6.0, (4.0, 0.2))])
def test_few_rays_are_those_of_many(extent, levels):
    import torch
    import paper_2402_13747_amd as pcrl
    s = _stretched(extent)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)))
    o, d = _rays(torch, s, 4097)
    tr = torch.tensor([[0.3, 4.0]]).expand(4097, 2).contiguous().cuda()
    for kw in (lambda a, b: {}, lambda a, b: dict(t_range=tr[a:b])):
        every = pcrl.sdf_intersect(scene, o, d, **kw(0, 4097))
        for a, b in [(i, i + 1) for i in range(40)] + [(40, 48), (48, 57), (0, 63), (1, 4097)]:
            few = pcrl.sdf_intersect(scene, o[a:b], d[a:b], **kw(a, b))
            _same({k: every[k][a:b] for k in ("t", "point", "normal", "leaf_cell")}, few)
    # rays that meet nothing: no direction, not a number, an empty range
    bad = pcrl.sdf_intersect(scene, o[:3], torch.tensor([[0.0, 0, 0], [float("nan"), 0, 1], [float("inf"), 0, 0]], device="cuda"))
    assert torch.isinf(bad["t"]).all() and (bad["leaf_cell"] == -1).all()
