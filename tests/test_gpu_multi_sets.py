"""Merged cluster sets, a set's workgroups of its own: one set, a number that
does not divide the grid, and the most a call takes, with sets of no cluster
first, last and between, one of a single point and one that dwarfs the rest --
each set exactly what it gets alone."""
import numpy as np
import pytest

from tests.gpu_util import hulls_np, note, planes_np, ragged_clusters
from tests.test_gpu_fused import SEED, _run, _same, _view

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7, 16])
def test_each_set_as_alone(n):
    import torch
    import paper_2510_01592_amd as vm
    H = 64
    empty = (np.zeros(1, np.uint32), np.zeros((0, 3), np.float32), np.zeros(0, np.uint32))
    point = (np.array([0, 1], np.uint32), np.ones((1, 3), np.float32), np.array([4], np.uint32))
    data = []
    for i in range(n):
        if n > 1 and i in (0, 3, n - 1):
            data.append(empty)
        elif i == 5:
            data.append(point)
        else:
            data.append(ragged_clusters(seed=60 + i, n_clusters=6, n_max=60_000 if i == 2 else 3_000))
    # (a view of no cluster still needs memory behind its pointers)
    pad = lambda d: (d[0], d[1] if len(d[1]) else np.zeros((1, 3), np.float32), d[2] if len(d[2]) else np.zeros(1, np.uint32))
    views = [_view(vm, *d) if len(d[2]) else _empty_view(vm, pad(d)) for d in data]
    Ks, Ns = [max(len(d[2]), 1) for d in data], [max(len(d[1]), 1) for d in data]
    work = torch.empty(vm.multi_workspace_bytes(sum(Ks), sum(Ns), H), dtype=torch.uint8, device="cuda")
    pbs = [vm.PlaneBuffers.alloc(K, N, H, with_all=True) for K, N in zip(Ks, Ns)]
    hbs = [vm.HullBuffers.alloc(K, N) for K, N in zip(Ks, Ns)]
    note(f"multi sets {n}")
    vm.planes_hulls_multi([v for v, _ in views], list(range(n)), vm.ransac_params(H, 0.01, SEED, 0), pbs, hbs, sum(Ks),
                          sum(Ns), work)
    torch.cuda.synchronize()
    for i, (cl, _) in enumerate(views):
        got = planes_np(pbs[i]), hulls_np(hbs[i])
        assert got[0]["status"] == 0 and got[1]["status"] == 0
        if len(data[i][2]) == 0:
            assert got[0]["in_off"][0] == 0 and got[1]["v_off"][0] == 0
        else:
            _same(got, _run(vm, cl, H, i, False), len(data[i][2]))


def _empty_view(vm, d):
    import torch
    view, keep = _view(vm, np.array([0, len(d[1])], np.uint32), d[1], d[2])
    meta = torch.zeros(2, dtype=torch.int32, device="cuda")
    view.d_meta = meta.data_ptr()
    return view, (keep, meta)
