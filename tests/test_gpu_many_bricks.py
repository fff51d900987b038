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


@pytest.mark.parametrize("side,levels", [
    (2300, (192.0, 3.0, 1.0)),     # 5.3 M parents, a leaf each
    (8300, (192.0, 3.0, 1.0)),     # 68.9 M
])
def test_every_parent_is_walked_over(side, levels):
    """The implicit surface there (skip radii of every parent's leaf cells): rays straight down onto points, and slanted
    ones, whose walk crosses many parents before the point it ends at."""
    import torch
    import paper_2402_13747_amd as pcrl
    n = side * side
    i = torch.arange(n, device="cuda")
    xyz = 3.0 * torch.stack([(i % side).float(), (i // side).float(), torch.zeros(n, device="cuda")], 1)
    nrm = torch.tensor([0.0, 0.0, 1.0], device="cuda").expand(n, 3).contiguous()
    scene = pcrl.build_voxels(xyz, nrm, torch.zeros(n, dtype=torch.int32, device="cuda"), levels, 0.05)
    assert scene.info()["n_nodes"][1] >= n
    pick = torch.cat([torch.randint(0, n, (2000,), generator=torch.Generator().manual_seed(1)).cuda(), i[-64:], i[:64]])
    for d in ([0.0, 0.0, -1.0], [0.8, 0.0, -0.6]):
        d = torch.tensor(d, device="cuda").expand(len(pick), 3).contiguous()
        # 2.4 m before the point: above the points beside it all the way
        got = pcrl.sdf_intersect(scene, (xyz[pick] - 2.4 * d).contiguous(), d)
        assert (got["t"] - 2.4).abs().max() < 2e-3  # eps: 1e-3 leaf edges; and FP32 positions of 25 km
        assert got["point"][:, 2].abs().max() < 2e-3
    scene.release()
    torch.cuda.empty_cache()
