"""A launch of more cones than waves are launched for (2^22): each cone is marched, a transmitter's paths are those that it
has alone."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def test_more_cones_than_waves():
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room(h=0.1)
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, float(np.float32(s.surfel_radius)))
    voxel = 0.2
    lo, hi = np.asarray(s.xyz).min(0), np.asarray(s.xyz).max(0)
    origin = (np.floor(lo / voxel) * voxel - 0.73 * voxel).astype(np.float32)
    ies = pcrl.ie_build(scene, origin, voxel, 2, np.ceil((hi - origin) / voxel).astype(int) + 2)
    g = torch.Generator().manual_seed(2)
    tx = torch.tensor(lo + 0.4) + torch.tensor(hi - lo - 0.8) * torch.rand(255, 3, generator=g)
    rx = torch.tensor([[2.0, 3.0, 1.0], [8.1, 2.2, 1.9]])

    def rows(t):
        L = pcrl.cone_launch(ies, t.float().cuda(), rx.cuda(), 1)
        p = pcrl.cone_collect(L, kappa=1 << 20, capacity=1 << 20)
        return L.stats(), {k: p[k].cpu().numpy() for k in ("tx", "rx", "n_refl", "key", "count", "len_poly", "points")}

    st, every = rows(tx)
    assert st["cones"][1] > 1 << 22, st["cones"]
    for j in (0, 127, 253, 254):
        _, alone = rows(tx[j:j + 1])
        mine = every["tx"] == j
        assert mine.sum() > 4
        # a key's paths come in the order of their priorities, which depend on the transmitter's number: as sets
        for k in ("rx", "n_refl", "key", "count"):
            assert np.array_equal(every[k][mine], alone[k]), (j, k)

        def table(r, m):
            t = np.concatenate([r[k][m].reshape(m.sum(), -1).astype(np.float64) for k in ("rx", "n_refl", "key", "len_poly", "points")], 1)
            t = np.nan_to_num(t, nan=-1.0)
            return t[np.lexsort(t.T)]

        assert np.array_equal(table(every, mine), table(alone, np.ones(len(alone["rx"]), bool))), j
