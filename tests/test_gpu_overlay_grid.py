"""Dynamic points in scenes of every size: an overlay whose top grid lies as deep as the base's, or deeper, hits what one
scene of all points hits, and a handful of points takes memory by their number, not by the scene's grid."""
import numpy as np
import pytest

from tests import parity
from tests.test_gpu_walk import _stretched

pytestmark = pytest.mark.gpu

# extent, levels; how many levels of bricks lie between the top grid and the leaves' parents, in the base and in the overlay
SHAPES = [
    (6.0, (0.3,)),                        # single level
    (6.0, (1.0, 0.2)),                    # 0, 0
    (420.0, (32.0, 2.0, 0.2)),            # 0, 1
    (350.0, (32.0, 2.0, 1.0, 0.1)),       # 0, 2
    (150.0, (32.0, 4.0, 0.25, 0.05)),     # 1, 1
    (420.0, (32.0, 2.0, 0.5, 0.1)),       # 1, 2
    (950.0, (32.0, 2.0, 0.5, 0.1)),       # 2, 2
]


def _both(pcrl, extent, levels):
    """The scene with a sixth of its points moving, and one scene of all points (the same numbers)."""
    s = _stretched(extent)
    n = len(s.xyz)
    move = np.zeros(n, bool)
    move[:n - 8:6] = True     # the lone points at the corners stay: the grid is the same
    order = np.concatenate([np.flatnonzero(~move), np.flatnonzero(move)])
    xyz, nrm, lab = s.xyz[order], s.normal[order], s.label[order]
    k, r = int((~move).sum()), float(np.float32(s.surfel_radius))
    whole = pcrl.build_voxels(xyz, nrm, lab, levels, r, t_eps=1e-3)
    scene = pcrl.build_voxels(xyz[:k], nrm[:k], lab[:k], levels, r, t_eps=1e-3)
    assert scene.info()["origin"] == whole.info()["origin"] and scene.info()["dims"] == whole.info()["dims"]
    scene.update_points(np.arange(k, n), xyz[k:], nrm[k:], lab[k:])
    return s, whole, scene


def _log(L):
    return [x.cpu().numpy() for x in L.hit_log]


def _equal(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y, equal_nan=x.dtype.kind == "f")


@pytest.mark.parametrize("extent,levels", SHAPES)
def test_overlay_hits_what_one_scene_hits(extent, levels):
    import paper_2402_13747_amd as pcrl
    s, whole, scene = _both(pcrl, extent, levels)
    for kw in (dict(), dict(stats=True)):
        a, b = (pcrl.launch_rays(x, s.tx, s.rx, n_rays=3000, max_reflections=3, hit_log=True, **kw) for x in (whole, scene))
        _equal(_log(a), _log(b))
    dynamic = _log(b)[0] >= scene.info()["n_points"]
    assert dynamic.sum() > 100
    # batched, with a query of the other scene beside it
    la, lb = pcrl.launch_batch([dict(scene=x, tx=s.tx, rx=s.rx, n_rays=3000, max_reflections=3, hit_log=True)
                                for x in (whole, scene)])
    _equal(_log(la), _log(a))
    _equal(_log(lb), _log(a))
    # refined
    P = pcrl.collect_paths(a, kappa=20)
    ra, rb = (parity.to_numpy(pcrl.refine_paths(x, s.tx, s.rx, P)) for x in (whole, scene))
    for k in ("status", "iters", "point_id", "key", "kept", "points", "length", "grad"):
        assert np.array_equal(ra[k], rb[k], equal_nan=ra[k].dtype.kind == "f"), k


@pytest.mark.parametrize("extent,levels", [(790.0, (32.0, 2.0, 0.5, 0.1)), (790.0, (32.0, 2.0, 0.2))])
def test_a_handful_of_points_takes_little(extent, levels):
    """A grid of 61 M cells (0.5 GB) belongs to the base alone."""
    import paper_2402_13747_amd as pcrl
    s = _stretched(extent)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)))
    held = scene.info()["device_bytes"]
    assert held > 400_000_000
    p = s.xyz[:5] + np.float32(0.05)
    scene.update_points(np.arange(len(s.xyz), len(s.xyz) + 5), p, s.normal[:5], s.label[:5])
    assert scene.info()["device_bytes"] - held < 1_000_000
