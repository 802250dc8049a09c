"""The grouped insert's partition: calls at its threshold, around whole rows of
points and whole tiles, batches whose remainder is one point, one bucket or a
few, points outside the grid and NaN among them, one voxel that takes most of
the points, a pose, and points on cell borders -- the map exact against the
oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_map_equal, note

pytestmark = pytest.mark.gpu
T = 1 << 17


@pytest.mark.parametrize("n,batch", [(T - 1, 0), (T, 0), (T + 1, 17), (T + 513, 17), (2 * T + 1025, 17), (4 * T + 1, 18),
                                     (256 * 1024 + 1, 0), (1_000_003, 0), (3 * T, 16)])
@pytest.mark.parametrize("kind", ["room", "one voxel", "borders"])
def test_map_equals_the_oracle(n, batch, kind):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(n)
    s, dims = 0.01, (101, 97, 45)
    origin = (-0.2, 0.1, -0.3)
    if kind == "borders":
        p = rng.integers(-2, 103, size=(n, 3)) * s + origin
    else:
        p = rng.uniform(-0.05, 1.05, (n, 3)) * (np.array(dims) * s) + origin
        if kind == "one voxel":
            p[rng.random(n) < 0.9] = np.array(origin) + 0.555
    p = p.astype(np.float32)
    p[:: 997] = np.nan
    c, si = np.cos(0.2), np.sin(0.2)
    R = None if kind == "borders" else np.array([[c, -si, 0.0], [si, c, 0.0], [0.0, 0.0, 1.0]])
    t = None if kind == "borders" else np.array([0.01, -0.02, 0.003])
    om = oracle.OracleMap(origin, s, dims)
    m = vm.Map(origin, s, dims, 20, insert_batch_log2=batch)
    note(f"insert rows {n} batch {batch} {kind}")
    for part in (p, p[: T + 7]):
        om.insert(part, R, t)
        m.insert(torch.from_numpy(part).cuda(), R, t)
    torch.cuda.synchronize()
    assert_map_equal(m, om)
    m.close()
