"""The cast's line walk at its edges: grids whose cube edge is 2, 4, 8 and 16
cells and whose last cubes are ragged, single-cell-wide grids, lines shorter
than, equal to and beyond one round of lanes, partial waves of points, and
points far enough away for the 64-bit walk -- exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_map_equal, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,n", [((37, 23, 11), 63), ((1, 1, 200), 65), ((200, 1, 3), 1), ((131, 97, 70), 1500),
                                    ((403, 398, 201), 1100), ((700, 690, 330), 1025), ((1030, 1200, 560), 700)])
def test_lines_on_grids_of_every_cube_edge(dims, n):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(sum(dims) + n)
    s = 0.01
    hi = s * np.array(dims)
    m, om = vm.Map((0.0, 0.0, 0.0), s, dims, 18), oracle.OracleMap((0.0, 0.0, 0.0), s, dims)
    blob = rng.uniform(0, hi, size=(60_000, 3))
    t = hi * rng.uniform(0.3, 0.7, size=3)
    blob[::3] = t + (blob[::3] - t) * 0.2   # dense about the sensor
    blob = blob.astype(np.float32)
    pts = rng.uniform(-0.2 * hi, 1.2 * hi, size=(n, 3))
    pts[::5] = t + rng.normal(0, 0.2, size=pts[::5].shape)      # short lines
    pts[1::9] = t + rng.normal(0, 1, size=pts[1::9].shape) * 3e5   # dm beyond 2^24 voxels
    note(f"clearing lines {dims} n={n}")
    for step in range(2):
        for x in (m, om):
            x.insert(torch.from_numpy(blob).cuda() if x is m else blob)
        ps = (pts - t).astype(np.float32)
        m.clear_rays(torch.from_numpy(ps).cuda(), None, t)
        om.clear_rays(ps, np.eye(3), t)
        assert_map_equal(m, om)
