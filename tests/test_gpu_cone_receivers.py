"""Cones: a receiver's paths do not depend on how many receivers share the launch (they are tested 64 at a time), nor
on how far the cones march (64 voxels at a time)."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("voxel", [1.0, 0.5, 0.1])   # 0.1 m: marches of more than 64 voxels
@pytest.mark.parametrize("n_rx", [64, 65, 130])
def test_paths_do_not_depend_on_the_other_receivers(voxel, n_rx):
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    scene = pcrl.build_voxels(s.xyz, s.normal, s.label, s.levels, float(np.float32(s.surfel_radius)))
    g = torch.Generator().manual_seed(n_rx)
    lo, hi = np.asarray(s.xyz).min(0), np.asarray(s.xyz).max(0)
    rx = torch.tensor(lo + 0.4) + torch.tensor(hi - lo - 0.8) * torch.rand(n_rx, 3, generator=g)
    origin = (np.floor(lo / voxel) * voxel - 0.73 * voxel).astype(np.float32)
    dims = np.ceil((hi - origin) / voxel).astype(int) + 2
    ies = pcrl.ie_build(scene, origin, voxel, 2, dims)

    def rows(r):
        p = pcrl.cone_collect(pcrl.cone_launch(ies, s.tx, r.float().cuda(), 1), kappa=1 << 20)
        return {k: p[k].cpu().numpy() for k in ("rx", "n_refl", "key", "count", "len_poly", "points")}

    every = rows(rx)
    for j in sorted({0, 1, 62, 63, n_rx - 2, n_rx - 1}):
        alone, mine = rows(rx[j:j + 1]), every["rx"] == j
        assert mine.any()
        for k in ("n_refl", "key", "count", "len_poly", "points"):
            assert np.array_equal(every[k][mine], alone[k], equal_nan=alone[k].dtype.kind == "f"), (j, k)
