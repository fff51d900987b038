"""Default tile size of a batch: every query traces as it does alone, from batches whose rays leave
most waves idle (64-slot tiles) to those that fill them several times over (larger tiles)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rays", [1, 63, 65, 4_000, 1_500_000])
def test_default_tile_matches_solo(rays):
    import torch
    import paper_2402_13747_amd as pcrl
    import scenes
    s = scenes.box_room()
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, s.surfel_radius)
    qs = [dict(scene=scene, tx=s.tx, rx=s.rx, n_rays=n, max_reflections=1) for n in (rays, 64, 2 * rays + 1)]
    batch = pcrl.launch_batch(qs, waves_per_cu=1)
    for q, b in zip(qs, batch):
        solo = pcrl.launch_rays(**q)
        x, y = (pcrl.collect_paths(l, kappa=100, capacity=1 << 16) for l in (solo, b))
        assert x["n_rows"] == y["n_rows"] and solo.stats()["segments"] == b.stats()["segments"]
        for k in ("ray", "count", "len_poly", "len_unf"):
            assert torch.equal(x[k], y[k]), k
