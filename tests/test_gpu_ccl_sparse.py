"""Labelling of grids with few voxels a tile, where the face kernel leaves empty
tiles at once, and of one on each side of the line: clouds of a few voxels, blobs across faces,
edges and corners of tiles, a diagonal through every tile corner, lines along
each axis, and tiles with one voxel beside empty ones -- labels and clusters
exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import note

pytestmark = pytest.mark.gpu


def _fills(dims, rng):
    d = np.array(dims)
    n = int(d.max())
    yield "scattered", rng.integers(0, d, (300, 3))
    yield "blobs", (rng.integers(0, d, (25, 1, 3)) + rng.integers(-3, 4, (25, 90, 3))).reshape(-1, 3)
    c = np.stack(np.meshgrid(*(np.arange(0, k + 1, t) for k, t in zip(dims, (32, 16, 16))), indexing="ij"), -1).reshape(-1, 3)
    yield "tile corners", (c[:, None] + np.array([[0, 0, 0], [-1, -1, -1]])).reshape(-1, 3)
    yield "tile corners, the other diagonal", (c[:, None] + np.array([[-1, 0, 0], [0, -1, -1]])).reshape(-1, 3)
    t = np.arange(n)
    yield "diagonal", np.c_[t, t, t]
    yield "lines", np.concatenate([np.c_[t, 0 * t + 15, 0 * t + 16], np.c_[0 * t + 31, t, 0 * t + 3], np.c_[0 * t + 64, 0 * t + 1, t]])
    yield "one voxel", d[None] - 1
    # 64 voxels a tile, counting the tile rows of all eight dies: one less, and as many
    tiles = 8 * -(-dims[0] // 32) * -(-(-(-dims[1] // 16) * -(-dims[2] // 16)) // 8)
    cells = rng.choice(int(np.prod(d)), min(64 * tiles, int(np.prod(d))), replace=False)
    cells = np.c_[cells % dims[0], cells // dims[0] % dims[1], cells // (dims[0] * dims[1])]
    yield "below the line", cells[:-1]
    yield "at the line", cells


@pytest.mark.parametrize("dims", [(97, 66, 65), (129, 40, 100), (33, 200, 48), (64, 16, 700)])
def test_sparse_labels_equal_the_oracle(dims):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(sum(dims))
    s = 0.01
    for name, idx in _fills(dims, rng):
        idx = np.unique(idx[np.all((idx >= 0) & (idx < np.array(dims)), axis=1)], axis=0)
        pts = np.ascontiguousarray((idx + 0.5) * s, dtype=np.float32)
        om = oracle.OracleMap((0.0, 0.0, 0.0), s, dims)
        om.insert(pts)
        ref = oracle.ccl26(om.key, om.dims)[0]
        c = oracle.group(om.key, ref, om.means(), 2)
        m = vm.Map((0.0, 0.0, 0.0), s, dims, 18)
        m.insert(torch.from_numpy(pts).cuda())
        lab = torch.zeros(len(om.key), dtype=torch.int32, device="cuda")
        note(f"ccl sparse {dims} {name}")
        cl = m.ccl(2, labels=lab)
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), ref), name
        got = vm.read_clusters(cl)
        assert np.array_equal(got["off"], c.off) and np.array_equal(got["tag"], c.tag), name
        assert np.array_equal(got["key"], c.key), name
        m.close()
