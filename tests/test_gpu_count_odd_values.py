"""Inlier counting over the whole range of floats: points with subnormal, huge,
infinite and NaN coordinates among ordinary ones, thresholds that are subnormal,
below and above the line of the scaled test (2^-90), huge and infinite -- the
counts, planes and winners exact against the oracle, in clusters for one wave
and for the tiles, in both forms.  A hypothesis drawn from an infinite or a NaN
point has no plane: the library counts it as degenerate (-1), the oracle's steps
give it a NaN plane that no point is near (0); those are not compared further."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits, cluster_tensors, note

pytestmark = pytest.mark.gpu


def _clusters(rng):
    parts = []
    for n in (3, 40, 200, 256, 257, 700, 5000):
        for scale in (1.0, 1e-38, 1e-41, 1e20, 1e30, 3e38):
            p = np.c_[rng.uniform(-1, 1, (n, 2)), rng.normal(0, 0.05, n)]
            with np.errstate(all="ignore"):
                p[:: 3] *= scale
                p = p.astype(np.float32)
            if n >= 40:
                p[5, 0], p[9, 1], p[13, 2], p[17] = np.inf, -np.inf, np.nan, np.inf
            parts.append(p)
    # all of them subnormal: distances of a few units in the last place
    for n in (64, 900):
        parts.append((rng.integers(-40, 41, (n, 3)) * np.array([1, 1, 0]) * 1.4e-45 + rng.integers(-2, 3, (n, 3)) * 1.4e-45)
                     .astype(np.float32))
    off = np.zeros(len(parts) + 1, np.uint32)
    off[1:] = np.cumsum([len(p) for p in parts])
    return off, np.concatenate(parts), np.arange(len(parts), dtype=np.uint32) * 29 + 3


@pytest.mark.parametrize("eps", [1.4e-45, 1e-40, 1.1754944e-38, float(np.float32(2.0 ** -91)), 2.0 ** -90, 1e-20, 0.02, 1e25,
                                 3.4028235e38, float("inf")])
def test_counts_equal_the_oracle(eps):
    import torch
    import paper_2510_01592_amd as vm
    H = 150
    off, xyz, tag = _clusters(np.random.default_rng(12))
    K, N = len(tag), len(xyz)
    T = cluster_tensors(off, xyz, tag)
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    work = torch.empty(vm.workspace_bytes(K, N, H), dtype=torch.uint8, device="cuda")
    prm = vm.ransac_params(H, eps, 0x5EED, 3)
    ref = [oracle.ransac(xyz[a:b, 0], xyz[a:b, 1], xyz[a:b, 2], H, eps, 0x5EED, int(t), 3)
           for a, b, t in zip(off[:-1], off[1:], tag)]
    for form in ("two-pass", "persistent"):
        note(f"odd values {form} eps={eps}")
        pb = vm.PlaneBuffers.alloc(K, N, H, with_all=True)
        if form == "persistent":
            vm.planes_hulls(cl, prm, pb, vm.HullBuffers.alloc(K, N), work)
        else:
            vm.ransac_planes(cl, prm, pb, work)
        torch.cuda.synchronize()
        counts, best, hyp = pb.counts.cpu().numpy(), pb.best_h.cpu().numpy(), pb.hyp.cpu().numpy()
        in_off, in_idx = pb.in_off.cpu().numpy(), pb.in_idx.cpu().numpy()
        for k, r in enumerate(ref):
            plane = np.isfinite(r.hyp).all(axis=1)
            assert np.array_equal(counts[k][plane], r.counts[plane]), (form, k)
            assert np.array_equal(bits(hyp[k][plane]), bits(r.hyp[plane])), (form, k)
            assert np.all(r.counts[~plane] <= 0) and np.all(counts[k][~plane] <= 0), (form, k)
            if r.counts.max() > 0:
                assert best[k] == r.best_h, (form, k)
                assert np.array_equal(in_idx[in_off[k]:in_off[k + 1]], r.inliers), (form, k)
