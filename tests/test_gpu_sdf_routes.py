"""The implicit surface: a ray's intersection does not depend on how its leaves are marched (on one lane, or
handed out over a wave) nor on how a sample's points are found (dense prefixes or the bricks' masks)."""
import numpy as np
import pytest

import scenes
from tests.test_gpu_walk import _stretched

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2402_13747_amd as pcrl
    return torch, pcrl


def _rays(torch, s, n):
    """Rays from inside the scene's box (eight lone points apart); every other one skims a face of it."""
    g = torch.Generator().manual_seed(11)
    lo, hi = torch.tensor(s.xyz[:-8].min(0)), torch.tensor(s.xyz[:-8].max(0))
    o = lo + (hi - lo) * torch.rand(n, 3, generator=g)
    d = torch.randn(n, 3, generator=g)
    axis, face = torch.randint(3, (n,), generator=g), torch.randint(2, (n,), generator=g)
    near = torch.where(face == 0, lo[axis] + 0.03, hi[axis] - 0.03)
    skim = torch.arange(n) % 2 == 0
    rows = torch.arange(n)[skim]
    o[rows, axis[skim]] = near[skim]
    d[rows, axis[skim]] *= 0.01
    return o.cuda(), d.cuda()


def _same(a, b):
    for k in ("t", "point", "normal", "leaf_cell"):
        assert np.array_equal(a[k].cpu().numpy(), b[k].cpu().numpy(), equal_nan=k != "leaf_cell"), k


@pytest.mark.parametrize("extent,levels,compact", [
    (6.0, (0.3,), False), (6.0, (0.9, 0.3), False), (6.0, (0.9, 0.3), True), (6.0, (1.0, 0.2), False),
    (6.0, (2.0, 1.0, 0.2), False), (6.0, (4.0, 2.0, 1.0, 0.2), True),
    (420.0, (32.0, 2.0, 0.5, 0.1), False),   # no dense grid of the leaves' parents: points found through the masks
    (950.0, (32.0, 1.0, 0.25), False),
])
def test_intersections_do_not_depend_on_the_march(env, extent, levels, compact):
    torch, pcrl = env
    s = _stretched(extent)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), compact=compact)
    o, d = _rays(torch, s, 4200)
    for n in (1, 63, 4096, 4097, 4200):  # up to 4096 rays: a wave each; above: those with many samples
        one = pcrl.sdf_intersect(scene, o[:n], d[:n], with_stats=True)  # counted: one lane per ray
        _same(one, pcrl.sdf_intersect(scene, o[:n], d[:n]))
    tr = torch.tensor([[0.5, 3.0]]).expand(4200, 2).contiguous().cuda()
    _same(pcrl.sdf_intersect(scene, o, d, t_range=tr, with_stats=True), pcrl.sdf_intersect(scene, o, d, t_range=tr))


@pytest.mark.parametrize("levels", [(0.3,), (1.0, 0.2), (2.0, 1.0, 0.2)])
def test_launches_do_not_depend_on_the_march(env, levels):
    torch, pcrl = env
    s = scenes.random_scene(7, tilt_sigma=0.03, pos_sigma=0.002, n_tx=1, n_rx=3)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)))
    d = torch.nn.functional.normalize(torch.randn(9000, 3, generator=torch.Generator().manual_seed(5)), dim=1).cuda()
    logs = []
    for n in (4000, 9000):  # a wave per ray, and lanes
        L = pcrl.launch_rays(scene, s.tx, s.rx, n_rays=n, directions=d[:n].contiguous(), max_reflections=3, hit_log=True, sdf=True)
        logs.append([x.cpu().numpy().reshape(n, -1)[:4000] for x in L.hit_log])
    for a, b in zip(*logs):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
