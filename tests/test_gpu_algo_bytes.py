"""Algorithmic bytes of a launch, counted by hand: rays that start inside the leaf of the one disk that they hit, at every
depth of the top grid."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 50


@pytest.mark.parametrize("extent,levels,bytes_down", [
    (80.0, (0.8,), 8),                              # top cell, the leaf itself
    (40.0, (1.0, 0.2), 8 + 16),                     # top cell, block
    (420.0, (32.0, 2.0, 0.5, 0.1), 8 + 12 + 4 + 16),       # top cell, one brick word, the parent's box, block
    (950.0, (32.0, 2.0, 0.5, 0.1), 8 + 2 * 12 + 4 + 16),   # two brick words
])
def test_bytes_of_one_leaf(extent, levels, bytes_down):
    import paper_2402_13747_amd as pcrl
    h, r_s = levels[-1], levels[-1] / 10
    corners = np.array([[x, y, z] for x in (0, 1) for y in (0, 1) for z in (0, 1)], np.float32) * np.float32(extent)
    up = np.tile(np.float32([[0, 0, 1]]), (8 + N, 1))

    def build(xyz):
        n = len(xyz)
        return pcrl.build_voxels(xyz, up[:n], np.zeros(n, np.uint32), levels, r_s, t_eps=1e-4 * h)

    org = np.array(build(corners).info()["origin"], np.float64)
    # disks in the middle of leaves on a diagonal, each ray's origin a quarter of a leaf below its disk
    cells = 3 + np.linspace(0.1, 0.9, N)[:, None] * (extent / h) * np.ones(3)
    p = (org + (np.floor(cells) + 0.5) * h).astype(np.float32)
    scene = build(np.concatenate([corners, p]))
    assert np.allclose(scene.info()["origin"], org)
    tx = p - np.float32([0, 0, 0.25 * h])
    L = pcrl.launch_rays(scene, tx, np.zeros((0, 3), np.float32), n_rays=1, max_reflections=0, stats=True,
                         directions=np.float32([[0, 0, 1]]))
    st = L.stats()
    assert st["hits"] == st["leaves_visited"] == st["surfel_tests"] == N
    assert st["algo_bytes"] == N * (bytes_down + 8 + 32)
