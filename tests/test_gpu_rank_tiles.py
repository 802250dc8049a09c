"""Ranks and keys by tiles of 256 occupancy words: grids of one cell, at and
around one tile, and on both sides of the number of tiles whose totals a
workgroup of their own scans; empty, a few cells at the ends, random cells and
full rows -- exported keys against the cells set."""
import numpy as np
import pytest

from tests.gpu_util import export_np, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1), (31, 1, 1), (8191, 1, 1), (8192, 1, 1), (8193, 1, 1), (128, 64, 3),
                                  (512, 256, 256), (512, 256, 257)])
def test_keys_are_the_cells(dims):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(dims[0])
    n = int(np.prod(dims, dtype=np.int64))
    full = np.arange(max(0, n // 2 - 20_000), min(n, n // 2 + 20_000))
    ends = np.unique(np.clip([0, 1, 31, 32, 8191, 8192, n - 8193, n - 33, n - 32, n - 2, n - 1], 0, n - 1))
    m = vm.Map((0.0, 0.0, 0.0), 1.0, dims, 18)
    for name, keys in (("empty", np.zeros(0, np.int64)), ("ends", ends), ("full rows", full),
                       ("random", np.unique(rng.integers(0, n, size=min(n, 60_000))))):
        m.clear()
        note(f"rank tiles {dims} {name}")
        if len(keys):
            c = np.stack([keys % dims[0], keys // dims[0] % dims[1], keys // (dims[0] * dims[1])], 1)
            m.insert(torch.from_numpy(np.ascontiguousarray(c + 0.5, dtype=np.float32)).cuda())
        key, cnt, _, _ = export_np(m)
        assert np.array_equal(key.astype(np.int64), keys), name
        assert np.all(cnt == 1)
    m.close()
