"""Clusters with straight edges full of points: lattices whose cells repeat, flat
and under planes that tilt (the edges' points then differ by 1e-6 m in the
plane, and coincident points meet at the corners).  Vertex lists exact against
the oracle, and the hull stage within ten times what it takes for as many points
spread over a patch: with a corner of the filter polygon lost, or its extremes
compared too coarsely, all edge points are left to one thread (20 to 80 times)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits, cluster_tensors, hulls_np, note, planes_np

pytestmark = pytest.mark.gpu


def _hulls(vm, torch, xyz, tag, n_hyp=16):
    """plane and polygon of one cluster and the least time of the hull stage in microseconds"""
    T = cluster_tensors(np.array([0, len(xyz)], np.uint32), xyz, np.array([tag], np.uint32))
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    N = len(xyz)
    pb, hb = vm.PlaneBuffers.alloc(1, N, n_hyp), vm.HullBuffers.alloc(1, N)
    work = torch.empty(vm.workspace_bytes(1, N, n_hyp), dtype=torch.uint8, device="cuda")
    vm.ransac_planes(cl, vm.ransac_params(n_hyp), pb, work)
    times = []
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        vm.hulls(cl, pb, hb, work)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return planes_np(pb), hulls_np(hb), min(times)


@pytest.mark.parametrize("side,n,count", [(60, 6666, 60), (150, 60_000, 12), (400, 600_000, 4)])
def test_edges_full_of_points(side, n, count):
    import torch
    import paper_2510_01592_amd as vm
    note(f"edges {side} x {count}")
    rng = np.random.default_rng(side)
    _, _, base = _hulls(vm, torch, np.c_[rng.random((n, 2)) * 0.01 * side, rng.normal(0, 0.002, n)].astype(np.float32), 1)
    worst = 0.0
    for t in range(count):
        p = np.c_[rng.integers(0, side, (n, 2)) * 0.01, rng.normal(0, 0.002, n)].astype(np.float32)
        P, H, us = _hulls(vm, torch, p, t * 7 + 1)
        inl = P["in_idx"][:P["in_off"][1]]
        ref = oracle.hull(p[inl, 0], p[inl, 1], p[inl, 2], P["plane"][0])
        assert np.array_equal(H["v_idx"][:H["v_off"][1]], inl[ref.idx]), (t, H["v_off"][1], len(ref.idx))
        assert np.array_equal(bits(H["v_xyz"][:H["v_off"][1]]), bits(ref.xyz)), t
        worst = max(worst, us)
    assert worst <= 10 * base, (worst, base)
