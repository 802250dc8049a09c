"""Grouping by a radix sort of cluster ids: cluster counts at, below and past
one digit (2048), far into the second, no cluster at all, and maps of one, a
few and more steps per tile, with small clusters among large ones and voxels of
none -- cluster offsets, tags, keys and points exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits, note

pytestmark = pytest.mark.gpu


def _pairs(n, dims, rng):
    """n separate pairs of cells, three cells apart in y and z and four in x"""
    at = np.stack(np.meshgrid(np.arange(0, dims[0] - 1, 4), np.arange(0, dims[1], 3), np.arange(0, dims[2], 3),
                              indexing="ij"), -1).reshape(-1, 3)
    at = at[rng.permutation(len(at))[:n]]
    assert len(at) == n
    return np.concatenate([at, at + [1, 0, 0]])


@pytest.mark.parametrize("case", ["none", "2047", "2048", "2049", "30000", "slabs", "slabs and pairs"])
def test_clusters_equal_the_oracle(case):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(len(case))
    s, dims, mc = 0.01, (192, 160, 96), 2
    if case == "none":
        idx, mc = _pairs(700, dims, rng), 3
    elif case.isdigit():
        idx = np.concatenate([_pairs(int(case), dims, rng)])
    else:
        # slabs four cells apart with every tenth cell missing: 1.6M cells, two steps per tile
        x, y, z = np.meshgrid(*(np.arange(n) for n in (192, 160, 96)), indexing="ij")
        occ = (z % 16 < 12) & (rng.random(x.shape) < 0.9) & (z < 80)
        idx = np.argwhere(occ)
        if case == "slabs and pairs":
            p = _pairs(2600, (192, 160, 10), rng) + [0, 0, 84]
            idx = np.concatenate([idx, p])
    pts = np.ascontiguousarray((idx + rng.uniform(0.1, 0.9, idx.shape)) * s, dtype=np.float32)
    om = oracle.OracleMap((0.0, 0.0, 0.0), s, dims)
    om.insert(pts)
    m = vm.Map((0.0, 0.0, 0.0), s, dims, 22)
    m.insert(torch.from_numpy(pts).cuda())
    note(f"group sort {case}")
    cl = m.ccl(mc)
    torch.cuda.synchronize()
    got = vm.read_clusters(cl)
    c = oracle.group(om.key, oracle.ccl26(om.key, om.dims)[0], om.means(), mc)
    if case.isdigit():
        assert len(c.tag) == int(case)
    assert got["K"] == len(c.tag)
    assert np.array_equal(got["off"], c.off) and np.array_equal(got["tag"], c.tag)
    assert np.array_equal(got["key"], c.key)
    assert np.array_equal(bits(np.c_[got["x"], got["y"], got["z"]]), bits(c.xyz))
    m.close()
