"""Scenes of very many leaves' parents: more than waves are launched for, and more than 2^26 (a launch of a wave for each
would hold 2^32 threads)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,levels", [
    (2300, (64.0, 1.0, 1.0)),       # 5.3 M parents
    (2300, (64.0, 2.0, 1.0)),
    (8300, (64.0, 1.0, 1.0)),       # 68.9 M
])
def test_every_parent_is_built(side, levels):
    import torch
    import paper_2402_13747_amd as pcrl
    n = side * side
    i = torch.arange(n, device="cuda")
    xyz = torch.stack([(i % side).float(), (i // side).float(), torch.zeros(n, device="cuda")], 1)
    nrm = torch.tensor([0.0, 0.0, 1.0], device="cuda").expand(n, 3).contiguous()
    # one disk a leaf: its box, the rounding pad included, stays inside
    scene = pcrl.build_voxels(xyz, nrm, torch.zeros(n, dtype=torch.int32, device="cuda"), levels, 0.05)
    info = scene.info()
    assert info["n_nodes"][2] >= n and (levels[1] == 2.0 or info["n_nodes"][1] == info["n_nodes"][2])
    # straight down onto disks all over the plane, the last ones included
    pick = torch.cat([torch.randint(0, n, (4000,), generator=torch.Generator().manual_seed(1)).cuda(), i[-64:], i[:64]])
    tx = xyz[pick] + torch.tensor([0.01, 0.01, 0.6], device="cuda")
    L = pcrl.launch_rays(scene, tx, torch.zeros((0, 3), device="cuda"), n_rays=1, max_reflections=0, hit_log=True,
                         directions=torch.tensor([[0.0, 0.0, -1.0]], device="cuda"))
    assert torch.equal(L.hit_log[0].reshape(-1).long(), pick)
    del L
    scene.release()
    torch.cuda.empty_cache()
