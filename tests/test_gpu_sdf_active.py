"""A launch over the implicit surface counts the rays that enter each segment: as many as its hit log holds there (a
segment that did not run is logged as -2), on lanes and on whole waves, and each a hit of the segment before."""
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coherent", [False, True])
@pytest.mark.parametrize("rays", [1, 100, 4096, 4097, 30_000])   # up to 4096 rays: a wave each
def test_active_is_the_hit_log(rays, coherent):
    import paper_2402_13747_amd as pcrl
    s = scenes.random_scene(7, tilt_sigma=0.03, pos_sigma=0.002, n_tx=2, n_rx=2)
    b = scenes.box_room()
    for c in (s, b):  # few rays go on; most do
        scene = pcrl.build_voxels(c.xyz, c.normal, c.label, c.levels, c.surfel_radius)
        L = pcrl.launch_rays(scene, c.tx, c.rx, n_rays=rays, max_reflections=4, hit_log=True, sdf=True, coherent=coherent)
        ids = L.hit_log[0].reshape(-1, 5)
        st = L.stats()
        want = [int((ids[:, k] != -2).sum()) for k in range(5)]
        assert list(st["active"][:5]) == want and st["segments"] == sum(want)
        assert want[1:] == [int((ids[:, k] >= 0).sum()) for k in range(4)]
