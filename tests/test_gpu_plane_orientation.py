"""Planes whose unit normal has no z component are oriented to +y, then +x:
points on a lattice give such planes exactly; every hypothesis' plane against
the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits, cluster_tensors, note

pytestmark = pytest.mark.gpu


def test_horizontal_normals_follow_the_tie_rule():
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(11)
    xyz = (rng.integers(-3, 4, size=(600, 3)) * 0.25).astype(np.float32)
    off, tag, H = np.array([0, 600], np.uint32), np.array([7], np.uint32), 512
    T = cluster_tensors(off, xyz, tag)
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    work = torch.empty(vm.workspace_bytes(1, 600, H), dtype=torch.uint8, device="cuda")
    pb = vm.PlaneBuffers.alloc(1, 600, H, with_all=True)
    note("plane orientation on a lattice")
    vm.ransac_planes(cl, vm.ransac_params(H, 0.1, 0x5EED, 3), pb, work)
    torch.cuda.synchronize()
    r = oracle.ransac(xyz[:, 0], xyz[:, 1], xyz[:, 2], H, 0.1, 0x5EED, 7, 3)
    assert (r.hyp[:, 2] == 0.0).sum() > 20   # the rule is reached
    assert np.array_equal(bits(pb.hyp[0].cpu().numpy()), bits(r.hyp))
