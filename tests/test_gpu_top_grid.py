"""Top grids whose skip codes are made in several turns (more than 4 M words of occupancy: thin grids and those of more
than 512 M cells): rays cross their empty cells and hit what they hit in a scene with a small top grid, and the codes
take no memory by the cell of a thin grid."""
import ctypes as C

import numpy as np
import pytest

from tests.test_gpu_sdf_alloc import Limited

pytestmark = pytest.mark.gpu


def _disks(size, n, seed):
    rng = np.random.default_rng(seed)
    xyz = (rng.uniform(0.02, 0.98, (n, 3)) * size).astype(np.float32)
    xyz[:8] = np.array([[x, y, z] for x in (0, 1) for y in (0, 1) for z in (0, 1)], np.float32) * np.float32(size)
    nrm = rng.normal(size=(n, 3)).astype(np.float32)
    return xyz, nrm, (np.arange(n) % 7).astype(np.uint32)


@pytest.mark.parametrize("size,flat,other", [
    ((6.0, 420.0, 420.0), (0.1,), (1.6, 0.1)),      # 1.1 G cells, 17.7 M words: five turns of rows
    ((0.5, 300.0, 300.0), (0.2, 0.1), (1.6, 0.1)),  # 9 x 1,501 x 1,501 parents
    ((3.0, 1600.0, 500.0), (0.2, 0.1), (1.6, 0.1)),  # 40 M parents of two leaves an axis, 20 M words
    ((420.0, 6.0, 420.0), (0.1,), (1.6, 0.1)),      # rows of 66 words
])
def test_hits_do_not_depend_on_the_turns(size, flat, other):
    import torch
    import paper_2402_13747_amd as pcrl
    size = np.array(size, np.float32)
    xyz, nrm, lab = _disks(size, 4000, 3)
    tx = (np.random.default_rng(5).uniform(0.05, 0.95, (6, 3)) * size).astype(np.float32)
    logs = []
    for levels in (flat, other):
        scene = pcrl.build_voxels(xyz, nrm, lab, levels, 1.0, t_eps=1e-3)
        L = pcrl.launch_rays(scene, tx, np.zeros((0, 3), np.float32), n_rays=20_000, max_reflections=2, hit_log=True)
        logs.append([x.cpu().numpy() for x in L.hit_log])
        del L
        scene.release()
    assert (logs[0][0][:, 0] >= 0).sum() > 2000
    for a, b in zip(*logs):
        assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f")
    torch.cuda.empty_cache()


def test_a_thin_grid_takes_no_memory_by_the_word():
    """The largest block that building a one-cell-thick grid asks for is one of its own size (8 B a cell), not the codes'
    224 B a word."""
    import torch
    import paper_2402_13747_amd as pcrl
    xyz, nrm, lab = _disks(np.float32([0.0, 900.0, 900.0]), 64, 3)
    most = []
    with Limited(torch, pcrl._lib) as A:
        fns = (pcrl._lib.ALLOC_FN(lambda size, stream, ctx: most.append(size) or A.alloc(size, stream, ctx)), A.fns[1])
        counted = pcrl._lib.PcrlAllocator(fns[0], fns[1], None)
        assert pcrl._lib.lib.set_allocator(C.byref(counted)) == 0
        scene = pcrl.build_voxels(xyz, nrm, lab, (0.2,), 0.05)
        cells = int(np.prod([int(x) for x in scene.info()["dims"]]))
        scene.release()
        torch.cuda.synchronize()
    assert cells > 60_000_000
    assert max(most) <= 1.5 * max(8 * cells, 224 << 22), max(most)
