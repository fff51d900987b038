"""Sorts that move values with their keys, at the sizes where the sort changes shape (one block, tiles of 2048 and of 8192
keys, a last tile of one key): the build's, of keys that leave no room for the point index, and the one of the
intersectable entities, which always moves values."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spread", [1, 3, 64])
@pytest.mark.parametrize("n", [513, 1023, 1025, 4095, 4096, 4097, 6145, 8192, (1 << 18), (1 << 18) + 1, 2_500_000])
def test_entries_with_their_ids(n, spread):
    import torch
    import paper_2402_13747_amd as pcrl
    g = torch.Generator(device="cuda").manual_seed(n)
    cell = torch.randint(0, spread, (n, 3), device="cuda", generator=g)
    cell[0], cell[-1] = 0, 1 << 14
    xyz = (cell + 0.5 + 0.2 * torch.rand((n, 3), device="cuda", generator=g)).float()
    nrm = torch.tensor([0.0, 0.0, 1.0], device="cuda").expand(n, 3).contiguous()
    scene = pcrl.build_voxels(xyz, nrm, torch.zeros(n, dtype=torch.int32, device="cuda"), (262144.0, 4096.0, 64.0, 1.0), 0.01)
    info = scene.info()
    # one coarsest cell (1 bit) and three levels of 64^3 (18 bits each): the point index does not fit below the key
    assert list(info["dims0"]) == [1, 1, 1] and info["key_bits"] == 55
    assert info["key_bits"] + int(n - 1).bit_length() > 64
    key, begin, count, ids = (x.cpu().numpy().astype(np.int64) for x in scene.leaf_table())
    assert (key[1:] > key[:-1]).all()
    assert begin[0] == 0 and (begin[1:] == begin[:-1] + count[:-1]).all() and begin[-1] + count[-1] == len(ids)
    assert np.array_equal(np.unique(ids), np.arange(n))
    # the sort is stable: leaf by leaf, ids ascend
    inner = np.ones(len(ids), bool)
    inner[begin] = False
    assert (ids[1:] > ids[:-1])[inner[1:]].all()
    # each entry's leaf holds its point or touches its disk
    c = np.floor((xyz.cpu().numpy() - np.asarray(info["origin"], np.float32)) / np.float32(info["leaf_size"]))
    leaf = np.repeat(np.arange(len(key)), count)
    assert np.abs(c[ids] - c[ids[begin]][leaf]).max() <= 2


@pytest.mark.parametrize("labels", [1, 5, 1 << 20])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1025, 2048, 4095, 4096, 4097, 8193, (1 << 18), (1 << 18) + 1])
def test_entities_are_grouped(n, labels):
    import torch
    import paper_2402_13747_amd as pcrl
    rng = np.random.default_rng(n)
    xyz = rng.uniform(0.1, 3.9, (n, 3)).astype(np.float32)
    lab = rng.integers(0, labels, n).astype(np.uint32)
    nrm = np.tile(np.float32([[0, 0, 1]]), (n, 1))
    scene = pcrl.build_voxels(xyz, nrm, lab, (1.0, 0.25), 0.01)
    t = pcrl.ie_build(scene, (0.0, 0.0, 0.0), 1.0, 2, (4, 4, 4)).table()
    sub = np.floor(xyz * np.float32(2.0)).astype(np.int64)
    vox, loc = sub // 2, sub % 2
    v = vox[:, 0] + 4 * (vox[:, 1] + 4 * vox[:, 2])
    w = loc[:, 0] + 2 * (loc[:, 1] + 2 * loc[:, 2])
    rows = np.stack([v, w, lab.astype(np.int64)], 1)
    want, first, inverse, count = np.unique(rows, axis=0, return_index=True, return_inverse=True, return_counts=True)
    assert np.array_equal(t["label"].cpu().numpy().astype(np.int64), want[:, 2])
    assert np.array_equal(t["count"].cpu().numpy().astype(np.int64), count)
    assert np.array_equal(t["sub"].cpu().numpy().reshape(-1, 3).astype(np.int64), sub[first])
    # the mean of each entity's positions, summed in FP64 and rounded to FP32: its points are the right ones
    mean = np.zeros((len(want), 3))
    np.add.at(mean, inverse.reshape(-1), xyz.astype(np.float64))
    mean /= count[:, None]
    assert np.abs(t["pos"].cpu().numpy()[:, :3] - mean).max() <= 4 * 2.0 ** -24 * 2
