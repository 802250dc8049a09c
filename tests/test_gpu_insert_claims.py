"""The small insert's claims: points into empty slots, into voxels that are
there, and into voxels cleared since (their slots keep the key with a count of
0), many points to a voxel and one, in a table that is nearly full of probe
chains -- the map exact against the oracle after each call, and the numbers of
occupied voxels and inserted points with it."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_map_equal, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,voxels", [(1, 1), (65, 1), (5000, 3), (20_000, 700), (60_000, 20_000), (131_071, 900)])
def test_new_present_and_cleared_voxels(n, voxels):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(n)
    s, dims, origin = 0.01, (64, 48, 40), (0.0, 0.0, 0.0)
    log2 = max(10, int(np.ceil(np.log2(voxels * 1.1))))
    m, om = vm.Map(origin, s, dims, log2), oracle.OracleMap(origin, s, dims)
    cells = rng.choice(int(np.prod(dims)), voxels, replace=False)
    cells = np.c_[cells % dims[0], (cells // dims[0]) % dims[1], cells // (dims[0] * dims[1])]
    note(f"insert claims {n} into {voxels}, table 2^{log2}")
    inserted = 0
    for step in range(3):
        p = ((cells[rng.integers(0, voxels, n)] + rng.random((n, 3)) * 0.98 + 0.01) * s).astype(np.float32)
        m.insert(torch.from_numpy(p).cuda())
        om.insert(p)
        inserted += n
        assert_map_equal(m, om)
        st = m.stats()
        assert (st.occupied, st.points_in, st.points_lost, st.status_flags) == (len(om.key), inserted, 0, 0)
        # free what lies along rays to the far faces
        t = np.array(dims) * s * 0.5
        r = (rng.uniform(-1, 1, (500, 3)) * np.array(dims) * s).astype(np.float32)
        m.clear_rays(torch.from_numpy(r).cuda(), None, t)
        om.clear_rays(r, np.eye(3), t)
        assert_map_equal(m, om)
    m.close()
