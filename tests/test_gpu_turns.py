"""Large launches deal their blocks out to the XCDs in turns: every ray is traced once, and hits what it hits in a
small launch."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, 1_200_003, 2_400_000])
def test_hits_do_not_depend_on_the_turns(n):
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.random_scene(3, tilt_sigma=0.02, n_rx=2)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, float(np.float32(s.surfel_radius)), t_eps=1e-3)
    d = torch.nn.functional.normalize(torch.randn(n, 3, generator=torch.Generator().manual_seed(5)), dim=1).cuda()

    def log(part):
        L = pcrl.launch_rays(scene, s.tx, s.rx, n_rays=len(part), max_reflections=1, directions=part.contiguous(),
                             ray_spacing=1e-3, hit_log=True)
        assert L.stats()["rays"] == len(part) * len(s.tx)
        return [x.reshape(len(s.tx), len(part), -1) for x in L.hit_log]

    ids, t = log(d)
    for a in range(0, n, 500_000):
        i, u = log(d[a:a + 500_000])
        assert torch.equal(i, ids[:, a:a + 500_000])
        assert torch.equal(u.nan_to_num(-1.0), t[:, a:a + 500_000].nan_to_num(-1.0))
