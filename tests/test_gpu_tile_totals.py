"""Grids and maps of so many scan tiles that a workgroup scans their totals: a
length that is no multiple of a read, and totals of more than one round (past
32768 tiles of grid words, past 16384 tiles of occupied voxels) -- exported keys
and clusters against the cells set."""
import numpy as np
import pytest

from tests.gpu_util import export_np, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(512, 257, 259), (1024, 512, 513)])
def test_ranks_past_one_read(dims):
    import torch
    import paper_2510_01592_amd as vm
    n = int(np.prod(dims, dtype=np.int64))
    rng = np.random.default_rng(7)
    keys = np.unique(np.r_[rng.integers(0, n, size=100_000), np.arange(n - 40, n)])
    c = np.stack([keys % dims[0], keys // dims[0] % dims[1], keys // (dims[0] * dims[1])], 1)
    m = vm.Map((0.0, 0.0, 0.0), 1.0, dims, 18)
    m.insert(torch.from_numpy(np.ascontiguousarray(c + 0.5, dtype=np.float32)).cuda())
    note(f"tile totals {dims}")
    assert np.array_equal(export_np(m)[0].astype(np.int64), keys)
    m.close()


def test_clusters_past_one_round():
    """Layers of 480 x 480 cells, every other layer empty, 100 layers (23M cells): a
    hash of 2^26 slots.  Every layer is one cluster; its tag is its first cell."""
    import torch
    import paper_2510_01592_amd as vm
    dims, layers = (480, 480, 200), 100
    m = vm.Map((0.0, 0.0, 0.0), 1.0, dims, 26)
    a = torch.arange(480, device="cuda", dtype=torch.float32) + 0.5
    y, x = torch.meshgrid(a, a, indexing="ij")
    for z in range(layers):
        m.insert(torch.stack([x, y, torch.full_like(x, 2 * z + 0.5)], -1).reshape(-1, 3).contiguous())
    note("tile totals: layers")
    cl = m.ccl(30)
    torch.cuda.synchronize()
    got = vm.read_clusters(cl)
    per = 480 * 480
    first = np.arange(layers, dtype=np.int64) * 2 * per
    assert got["K"] == layers
    assert np.array_equal(got["off"].astype(np.int64), np.arange(layers + 1) * per)
    assert np.array_equal(got["tag"].astype(np.int64), first)
    assert np.array_equal(got["key"].astype(np.int64), (first[:, None] + np.arange(per)).ravel())
    m.close()
