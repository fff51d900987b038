"""A refined path does not depend on how many lanes refine it (64, 32, 16 or 8, by the number of paths)."""
import numpy as np
import pytest

from tests.test_gpu_walk import _stretched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extent,levels,smooth", [
    (6.0, (0.3,), 0.0), (6.0, (1.0, 0.2), 0.0), (6.0, (1.0, 0.2), 0.95), (6.0, (2.0, 1.0, 0.2), 0.95),
    (420.0, (32.0, 2.0, 0.5, 0.1), 0.0),
])
def test_paths_do_not_depend_on_their_lanes(extent, levels, smooth):
    import torch
    import paper_2402_13747_amd as pcrl
    s = _stretched(extent)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), t_eps=1e-3)
    # coarse points anywhere in the scene: the rays towards them hit what they hit
    rows = [(i, j, k) for i in range(2) for j in range(4) for k in range(4) for _ in range(6)]
    n, g = len(rows), torch.Generator().manual_seed(2)
    lo, hi = torch.tensor(s.xyz[:-8].min(0)), torch.tensor(s.xyz[:-8].max(0))
    tx, rx, refl = (torch.tensor(x, dtype=torch.int32).cuda() for x in zip(*rows))
    P = dict(n_rows=n, tx=tx, rx=rx, n_refl=refl, points=(lo + (hi - lo) * torch.rand(n, 3, 3, generator=g)).cuda())
    kw = dict(max_iters=40, smooth_radius=smooth * scene.info()["leaf_size"])
    one = pcrl.refine_paths(scene, s.tx, s.rx, P, **kw)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    for waves in (1.5, 3.0, 6.0, 9.0):  # of the 12 that a CU holds at once, at 64 lanes a path; 9: a ragged last round
        m = int(waves * 12 * cu) // n + 1
        many = {k: v.repeat_interleave(m, 0).contiguous() if hasattr(v, "shape") else v for k, v in P.items()}
        many["n_rows"] = n * m
        r = pcrl.refine_paths(scene, s.tx, s.rx, many, **kw)
        for k in ("status", "iters", "grad", "length", "points", "point_id", "key"):
            a, b = one[k].repeat_interleave(m, 0).cpu().numpy(), r[k].cpu().numpy()
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), (k, m)
        assert r["n_kept"] == one["n_kept"]
