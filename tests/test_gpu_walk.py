"""The launcher's walk: every shape of its top grid and bricks finds the same hits, and so does every number
of rays per wave."""
import numpy as np
import pytest

import scenes
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2402_13747_amd as pcrl
    return torch, pcrl


def _stretched(extent):
    """A random scene in one corner of a cube of `extent`, spanned by eight lone points."""
    s = scenes.random_scene(7, tilt_sigma=0.03, pos_sigma=0.002, n_tx=2, n_rx=4)
    c = np.array([[x, y, z] for x in (0, 1) for y in (0, 1) for z in (0, 1)], np.float32) * extent
    s.xyz = np.concatenate([s.xyz, c]).astype(np.float32)
    s.normal = np.concatenate([s.normal, np.tile(np.float32([[0, 0, 1]]), (8, 1))])
    s.label = np.concatenate([s.label, np.full(8, 77, np.uint32)])
    return s


def _hits(pcrl, s, levels, rays=3000):
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), t_eps=1e-3)
    L = pcrl.launch_rays(scene, s.tx, s.rx, n_rays=rays, max_reflections=3, hit_log=True)
    p = parity.to_numpy(pcrl.collect_paths(L, kappa=1 << 30))
    return [x.cpu().numpy() for x in L.hit_log] + [np.asarray(p[k]) for k in ("ray", "key", "count", "len_poly")]


@pytest.mark.parametrize("extent,levels", [
    (6.0, (0.3,)), (6.0, (0.2, 0.2)), (6.0, (0.4, 0.2)), (6.0, (0.9, 0.3)), (6.0, (0.8, 0.2)), (6.0, (1.0, 0.2)),
    (40.0, (1.6, 0.1)), (40.0, (1.7, 0.1)), (40.0, (3.2, 0.1)), (40.0, (3.3, 0.1)), (40.0, (6.4, 0.1)),
    (6.0, (2.0, 1.0, 0.2)), (6.0, (4.0, 2.0, 1.0, 0.2)),
    (420.0, (32.0, 2.0, 0.5, 0.1)),   # the parents' grid would hold 600 M cells: the top grid is one level above
    (950.0, (32.0, 2.0, 0.5, 0.1)),   # and here two levels above
    (950.0, (32.0, 1.0, 0.25)),
])
def test_hits_do_not_depend_on_the_levels(env, extent, levels):
    torch, pcrl = env
    s = _stretched(extent)
    ref = _hits(pcrl, s, (extent / 40.0, extent / 400.0))
    got = _hits(pcrl, s, levels)
    for a, b in zip(ref, got):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")


@pytest.mark.parametrize("n", [1, 7, 65, 8 * 8192 - 1, 16 * 8192 + 15, 32 * 8192 + 40])
def test_hits_do_not_depend_on_rays_per_wave(env, n):
    """The first n of a fixed set of directions hit the same points whatever n is (8, 16, 32 or 64 rays a wave)."""
    torch, pcrl = env
    s = scenes.random_scene(3, tilt_sigma=0.02, n_rx=2)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, float(np.float32(s.surfel_radius)), t_eps=1e-3)
    d = torch.nn.functional.normalize(torch.randn(600_000, 3, generator=torch.Generator().manual_seed(5)), dim=1).cuda()

    def log(k):
        L = pcrl.launch_rays(scene, s.tx, s.rx, n_rays=k, max_reflections=2, directions=d[:k].contiguous(), hit_log=True)
        return L.hit_log

    ids, t = log(600_000)
    i, u = log(n)
    assert torch.equal(i, ids[:n]) and torch.equal(u.nan_to_num(-1.0), t[:n].nan_to_num(-1.0))
