"""Inlier counting on the matrix cores: every hypothesis' count and the winner
of clusters whose sizes straddle the 16-point steps, the 64-point rows, the
wave/tile split and the 4096-point tile, at hypothesis counts that straddle the
64-plane groups, the 256/512-plane chunks -- exact against the oracle, with
points that lie exactly at the threshold (strict: not counted) and with a
threshold too small for the scaled test (the comparing form)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits, cluster_tensors, note

pytestmark = pytest.mark.gpu
SIZES = (3, 15, 16, 17, 63, 64, 65, 200, 255, 256, 257, 273, 511, 513, 4095, 4096, 4097, 4161, 8193)


def _clusters():
    rng = np.random.default_rng(11)
    parts = []
    for i, n in enumerate(SIZES):
        if i % 2:
            # a quarter-unit lattice: many points at distance exactly 0 and exactly 0.25 of axis-aligned planes
            p = rng.integers(-3, 4, size=(n, 3)) * 0.25
        else:
            p = np.c_[rng.uniform(-1, 1, (n, 2)), rng.normal(0, 0.1, n)]
        parts.append(p.astype(np.float32))
    off = np.zeros(len(parts) + 1, np.uint32)
    off[1:] = np.cumsum([len(p) for p in parts])
    return off, np.concatenate(parts), np.arange(len(parts), dtype=np.uint32) * 31 + 1


@pytest.mark.parametrize("n_hyp", [1, 63, 65, 129, 257, 513])
@pytest.mark.parametrize("eps", [0.25, 0.01, 1e-30])
def test_counts_equal_the_oracle(n_hyp, eps):
    import torch
    import paper_2510_01592_amd as vm
    off, xyz, tag = _clusters()
    K, N = len(tag), len(xyz)
    T = cluster_tensors(off, xyz, tag)
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    work = torch.empty(vm.workspace_bytes(K, N, n_hyp), dtype=torch.uint8, device="cuda")
    prm = vm.ransac_params(n_hyp, eps, 0x5EED, 3)
    ref = [oracle.ransac(xyz[a:b, 0], xyz[a:b, 1], xyz[a:b, 2], n_hyp, eps, 0x5EED, int(t), 3)
           for a, b, t in zip(off[:-1], off[1:], tag)]
    for form in ("two-pass", "persistent"):
        note(f"matrix count {form} H={n_hyp} eps={eps}")
        pb = vm.PlaneBuffers.alloc(K, N, n_hyp, with_all=True)
        if form == "persistent":
            vm.planes_hulls(cl, prm, pb, vm.HullBuffers.alloc(K, N), work)
        else:
            vm.ransac_planes(cl, prm, pb, work)
        torch.cuda.synchronize()
        counts, best = pb.counts.cpu().numpy(), pb.best_h.cpu().numpy()
        for k, r in enumerate(ref):
            assert np.array_equal(counts[k], r.counts), (form, k, SIZES[k])
            assert best[k] == r.best_h, (form, k)
            assert np.array_equal(bits(pb.plane[k].cpu().numpy()), bits(r.plane)), (form, k)
