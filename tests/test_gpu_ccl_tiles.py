"""Labelling of tiles by their runs: grids at, below and past a tile's 32 x 16
x 16 cells and at every word offset, from sparse to full, alternate cells in x
(4096 runs in a tile), planes of alternate cells joined by one row, and combs
whose arms meet only at their far end -- labels and clusters exact against the
oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import note

pytestmark = pytest.mark.gpu


def _fills(dims, rng):
    x, y, z = np.meshgrid(*(np.arange(n) for n in dims), indexing="ij")
    for p in (0.02, 0.1, 0.3, 0.6, 0.97):
        yield f"random {p}", rng.random(dims) < p
    yield "full", np.ones(dims, bool)
    yield "alternate in x", x % 2 == 0
    yield "alternate in x, one row joins them", (x % 2 == 0) & (z % 2 == 0) | (y == dims[1] - 1) & (z == dims[2] - 1)
    yield "no two touch", (x % 2 == 0) & (y % 2 == 0) & (z % 2 == 0)
    yield "comb", (y % 2 == 0) | (x == dims[0] - 1)
    yield "comb in z", (z % 2 == 0) | (y == dims[1] - 1)
    yield "diagonals", (x + y + z) % 3 == 0
    yield "diagonals the other way", (x - y + 2 * z) % 5 == 0


@pytest.mark.parametrize("dims", [(32, 16, 16), (31, 15, 17), (33, 17, 16), (64, 32, 32), (65, 33, 18), (97, 16, 33),
                                  (1, 40, 40), (7, 3, 50), (130, 1, 20)])
def test_labels_equal_the_oracle(dims):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(sum(dims))
    s = 0.01
    for name, occ in _fills(dims, rng):
        idx = np.argwhere(occ)
        if len(idx) == 0:
            continue
        pts = np.ascontiguousarray((idx + 0.5) * s, dtype=np.float32)
        om = oracle.OracleMap((0.0, 0.0, 0.0), s, dims)
        om.insert(pts)
        m = vm.Map((0.0, 0.0, 0.0), s, dims, 18)
        m.insert(torch.from_numpy(pts).cuda())
        lab = torch.zeros(len(om.key), dtype=torch.int32, device="cuda")
        note(f"ccl tiles {dims} {name}")
        cl = m.ccl(3, labels=lab)
        torch.cuda.synchronize()
        ref = oracle.ccl26(om.key, om.dims)[0]
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), ref), name
        got = vm.read_clusters(cl)
        c = oracle.group(om.key, ref, om.means(), 3)
        assert np.array_equal(got["off"], c.off) and np.array_equal(got["tag"], c.tag), name
        assert np.array_equal(got["key"], c.key), name
        m.close()
