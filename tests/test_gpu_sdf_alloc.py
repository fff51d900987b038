"""Device memory that runs out while the first call over the implicit surface builds its index: the call reports it, the
scene stays as it was, and the next call gives the same intersections as in a scene that never ran out."""
import ctypes as C

import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


class Limited:
    """set_allocator from torch's caching allocator; `left` more blocks are given, then none."""

    def __init__(self, torch, lib):
        self.torch, self.lib, self.left, self.asked, self.sizes = torch, lib, 1 << 30, 0, {}
        self.fns = (lib.ALLOC_FN(self.alloc), lib.FREE_FN(self.free))
        self.a = lib.PcrlAllocator(self.fns[0], self.fns[1], None)

    def alloc(self, size, stream, ctx):
        self.asked += 1
        if self.left <= 0:
            return None
        self.left -= 1
        p = self.torch.cuda.caching_allocator_alloc(size, 0, stream or 0)
        self.sizes[p] = size
        return p

    def free(self, p, stream, ctx):
        if self.sizes.pop(p, None) is not None:
            self.torch.cuda.caching_allocator_delete(p)

    def __enter__(self):
        assert self.lib.lib.set_allocator(C.byref(self.a)) == 0
        return self

    def __exit__(self, *e):
        self.torch.cuda.synchronize()
        assert self.lib.lib.set_allocator(None) == 0


@pytest.mark.parametrize("levels,compact", [((0.25,), False), ((1.0, 0.25), False), ((1.0, 0.25), True), ((1.0, 0.5, 0.25), False)])
def test_index_that_runs_out_of_memory(levels, compact):
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    g = torch.Generator().manual_seed(3)
    o = (torch.tensor([[5.0, 4.0, 1.5]]) + torch.rand(500, 3, generator=g)).cuda()
    d = torch.randn(500, 3, generator=g).cuda()

    def build():
        return pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), compact=compact)

    ref = pcrl.sdf_intersect(build(), o, d)
    with Limited(torch, pcrl._lib) as A:
        scene = build()
        failed = 0
        for k in range(200):
            A.left = k
            try:
                got = pcrl.sdf_intersect(scene, o, d)
                break
            except Exception as e:
                assert "PCRL_ENOMEM" in str(e) or "allocation" in str(e), e
                failed += 1
        assert failed >= 5
        A.left = 1 << 30
        again = pcrl.sdf_intersect(scene, o, d)
        for x in (got, again):
            for k in ("t", "point", "normal", "leaf_cell"):
                assert torch.equal(torch.nan_to_num(ref[k].float(), 7.0), torch.nan_to_num(x[k].float(), 7.0)), k
        scene.release()
        torch.cuda.synchronize()
        assert not A.sizes  # nothing of the attempts is left


def test_ie_table_keeps_the_points_index_alone():
    """A table of intersectable entities leaves each point of the scene once (32 B) and 4 B per entry with it, not
    what only the implicit surface reads (blocks have less than half of slack)."""
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    with Limited(torch, pcrl._lib) as A:
        scene = pcrl.build_voxels(s.xyz, s.normal, s.label, (1.0, 0.1), float(np.float32(s.surfel_radius)))
        held = sum(A.sizes.values())
        info = scene.info()
        ies = pcrl.ie_build(scene, (-0.55, -0.45, -0.6), 0.5, 2, (23, 19, 9))
        assert ies.info()["n_ies"] > 100
        ies.release()
        torch.cuda.synchronize()
        kept = sum(A.sizes.values()) - held
        assert 32 * info["n_points"] <= kept <= 1.5 * (32 * info["n_points"] + 4 * info["n_entries"] + 1024), kept
        scene.release()
        torch.cuda.synchronize()
        assert not A.sizes


@pytest.mark.parametrize("levels", [(1.0, 0.1), (2.0, 1.0, 0.1)])
def test_compact_scene_keeps_no_table_of_leaf_cells(levels):
    """The implicit surface of a compact scene reads the bricks' masks: no table of the leaves' parents' cells, not even
    of prefixes (4 B a cell), is kept with the scene; a skip radius (1 B a cell) is."""
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    o = torch.tensor([[5.0, 4.0, 1.5]]).expand(200, 3).contiguous().cuda()
    d = torch.randn(200, 3, generator=torch.Generator().manual_seed(3)).cuda()
    kept, out = [], []
    for compact in (False, True):
        with Limited(torch, pcrl._lib) as A:
            scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), compact=compact)
            held = sum(A.sizes.values())
            out.append(pcrl.sdf_intersect(scene, o, d))
            torch.cuda.synchronize()
            kept.append(sum(A.sizes.values()) - held)
            parents, leaves = scene.info()["n_nodes"][len(levels) - 2:len(levels)]
            points, entries = scene.info()["n_points"], scene.info()["n_entries"]
            cells = 1000 * parents
            scene.release()
    assert kept[0] >= 12 * cells
    # per parent cell the skip radius and 4 B per 64 for the masks' child counts; the points' index
    assert kept[1] <= 1.5 * (1.1 * cells + 48 * points + 4 * entries + 4 * leaves + 64 * 1024), (kept, cells)
    for k in ("t", "point", "normal"):
        assert torch.equal(out[0][k].nan_to_num(-1.0, 1e30), out[1][k].nan_to_num(-1.0, 1e30)), k


@pytest.mark.parametrize("levels,compact", [((0.2,), False), ((1.0, 0.1), False), ((1.0, 0.1), True), ((2.0, 1.0, 0.1), False)])
def test_device_bytes_hold_the_index(levels, compact):
    """scene_info's device_bytes grow by the blocks that the scene's index keeps (each block is asked for rounded up by
    less than half, and to 512 bytes)."""
    import torch
    import paper_2402_13747_amd as pcrl
    s = scenes.box_room()
    o = torch.tensor([[5.0, 4.0, 1.5]]).cuda()
    with Limited(torch, pcrl._lib) as A:
        scene = pcrl.build_voxels(s.xyz, s.normal, s.label, levels, float(np.float32(s.surfel_radius)), compact=compact)
        for use in (lambda: pcrl.ie_build(scene, (-0.55, -0.45, -0.6), 0.5, 2, (23, 19, 9)).release(),
                    lambda: pcrl.sdf_intersect(scene, o, o)):
            held, said, blocks = sum(A.sizes.values()), scene.info()["device_bytes"], len(A.sizes)
            use()
            torch.cuda.synchronize()
            kept, grown = sum(A.sizes.values()) - held, scene.info()["device_bytes"] - said
            assert 0 < grown <= kept <= 1.5 * grown + 512 * (len(A.sizes) - blocks), (grown, kept)
        scene.release()
