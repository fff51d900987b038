"""Tiles of a batch: no tile size, the caller's or the autotuner's, leaves waves idle."""
import pytest

pytestmark = pytest.mark.gpu


def test_no_tile_leaves_waves_idle():
    """Few rays are dealt out in small tiles whatever tile the caller or the autotuner asks for: a batch of a thousand
    chunks of rays takes about as long with tiles of 1024 and 4096 slots, which alone would leave most waves idle and
    take several times as long, and with the autotuner's as by default.  Best of several runs each."""
    import time
    import torch
    import paper_2402_13747_amd as pcrl
    import scenes
    qs = []
    for seed in range(4):
        s = scenes.box_room()
        scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, s.surfel_radius)
        qs.append(dict(scene=scene, tx=s.tx, rx=s.rx, n_rays=200_000 >> seed, max_reflections=2))

    def best(**kw):
        for _ in range(3):
            pcrl.launch_batch(qs, **kw)
        times = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            L = pcrl.launch_batch(qs, **kw)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
            del L
        return min(times)

    base = best()
    for kw in (dict(tile_rays=1024), dict(tile_rays=4096), dict(autotune=True)):
        assert best(**kw) < 1.3 * base, kw
