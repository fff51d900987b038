"""The numbers of rays at which a launch changes between 8, 16 and 32 rays per wave: each ray hits what it hits in a large
launch."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8 * 4096 + 7, 8 * 4096 + 8, 16 * 4096 + 15, 16 * 4096 + 16, 32 * 8192 + 31, 32 * 8192 + 32])
@pytest.mark.parametrize("coherent", [False, True])
def test_hits_at_the_lines(n, coherent):
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.random_scene(3, tilt_sigma=0.02, n_rx=2)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, float(np.float32(s.surfel_radius)), t_eps=1e-3)
    d = torch.nn.functional.normalize(torch.randn(600_000, 3, generator=torch.Generator().manual_seed(5)), dim=1).cuda()

    def log(k):
        return pcrl.launch_rays(scene, s.tx[:1], None, n_rays=k, max_reflections=2, directions=d[:k].contiguous(), hit_log=True,
                                coherent=coherent).hit_log

    (ids, t), (i, u) = log(600_000), log(n)
    assert torch.equal(i, ids[:n]) and torch.equal(u.nan_to_num(-1.0), t[:n].nan_to_num(-1.0))
