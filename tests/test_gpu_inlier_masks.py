"""Inlier lists written from per-tile bit masks: cluster sizes around a mask
word, a wave and a tile, in an order that starts clusters at every offset
within a word, empty clusters between them, and a list capacity that ends
inside a cluster -- exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import cluster_tensors, note, planes_np

pytestmark = pytest.mark.gpu
SIZES = (3, 31, 0, 32, 33, 5, 63, 64, 65, 1, 127, 129, 2047, 0, 2049, 4095, 4, 4096, 7, 4097, 4127, 4129, 8191, 8193, 12289)


@pytest.mark.parametrize("cap_frac", [1.0, 0.5])
def test_lists_equal_the_oracle(cap_frac):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(5)
    off = np.zeros(len(SIZES) + 1, np.uint32)
    off[1:] = np.cumsum(SIZES)
    K, N, H = len(SIZES), int(off[-1]), 24
    xyz = np.c_[rng.uniform(-1, 1, (N, 2)), rng.normal(0, 0.012, N)].astype(np.float32)
    tag = np.arange(K, dtype=np.uint32) * 5 + 1
    T = cluster_tensors(off, xyz, tag)
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    cap = int(N * cap_frac)
    for form in ("two-pass", "persistent"):
        note(f"inlier masks {form} cap {cap}")
        work = torch.empty(vm.workspace_bytes(K, N, H), dtype=torch.uint8, device="cuda")
        pb, hb = vm.PlaneBuffers.alloc(K, cap, H, with_all=True), vm.HullBuffers.alloc(K, N)
        pb.in_idx.fill_(-1)
        prm = vm.ransac_params(H, 0.01, 0x5EED, 0)
        if form == "persistent":
            vm.planes_hulls(cl, prm, pb, hb, work)
        else:
            vm.ransac_planes(cl, prm, pb, work)
        torch.cuda.synchronize()
        P = planes_np(pb)
        want = []
        for k in range(K):
            a, b = int(off[k]), int(off[k + 1])
            r = oracle.ransac(xyz[a:b, 0], xyz[a:b, 1], xyz[a:b, 2], H, 0.01, 0x5EED, int(tag[k]), 0)
            assert int(P["in_off"][k]) == sum(len(w) for w in want), (form, k)
            assert P["best"][k] == r.best_h and P["nin"][k] == len(r.inliers), (form, k)
            want.append(r.inliers)
        want = np.concatenate(want)
        assert int(P["in_off"][K]) == len(want)
        n = min(cap, len(want))
        assert np.array_equal(P["in_idx"][:n], want[:n])
        assert (P["status"] != 0) == (len(want) > cap)
