"""A refined path does not depend on the room that its batch has for interactions (its state in LDS is laid out by it), at
every number of lanes per path."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 30, 60, 150])  # of 128 paths: 64, 32, 16 and 8 lanes each
@pytest.mark.parametrize("smooth", [0.0, 0.95])
def test_paths_do_not_depend_on_the_stride(copies, smooth):
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, float(np.float32(s.surfel_radius)))
    n = 128 * copies
    g = torch.Generator().manual_seed(copies)
    refl = torch.randint(0, 3, (n,), generator=g, dtype=torch.int32).sort().values.cuda()
    zero = torch.zeros(n, dtype=torch.int32, device="cuda")
    pts = (torch.tensor([10.0, 8.0, 3.0]) * torch.rand(n, 2, 3, generator=g)).cuda()
    kw = dict(max_iters=20, smooth_radius=smooth * scene.info()["leaf_size"])
    ref = None
    for K in (2, 3, 5, 8):
        points = torch.full((n, K, 3), float("nan"), device="cuda")
        points[:, :2] = pts
        r = pcrl.refine_paths(scene, s.tx, s.rx, dict(n_rows=n, tx=zero, rx=zero, n_refl=refl, points=points), **kw)
        r = {k: r[k].cpu().numpy() for k in ("status", "iters", "grad", "length", "points", "point_id", "key", "kept")}
        ref = ref or r
        assert (ref["status"] == 0).any()
        for k, a in ref.items():
            b = r[k][:, :2] if k in ("points", "point_id", "key") else r[k]
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (k, K)
    none = dict(n_rows=5, tx=zero[:5], rx=zero[:5], n_refl=zero[:5], points=torch.zeros((5, 0, 3), device="cuda"))
    assert (pcrl.refine_paths(scene, s.tx, s.rx, none, **kw)["status"] == 0).all()
