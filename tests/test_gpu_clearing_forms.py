"""Clearing in the grid's order (few rays) and in bricks (many): one ray less
than the bricks take and as many, on odd and thin grids, on one whose padded
cells need 64-bit addresses, in batches, captured before any call of many rays
and after -- the map exact against the oracle.  A call of few rays takes no more
memory than its two bitmaps."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_map_equal, note

pytestmark = pytest.mark.gpu


def _bricks_from(dims):
    """the number of rays from which a call walks bricks"""
    words = (int(np.prod([int(d) for d in dims])) + 31) // 32
    return -(-(6_000_000 + words + words // 4) // max(dims))


def _scene(rng, dims, s, n):
    """a map dense about the sensor, the sensor's place, and a frame's points from there"""
    hi = s * np.array(dims)
    t = hi * rng.uniform(0.3, 0.7, size=3)
    blob = rng.uniform(0, hi, size=(60_000, 3))
    blob[::3] = t + (blob[::3] - t) * 0.2
    pts = rng.uniform(-0.2 * hi, 1.2 * hi, size=(n, 3))
    pts[::5] = t + rng.normal(0, 0.2, size=pts[::5].shape)
    pts[1::997] = t + rng.normal(0, 1, size=pts[1::997].shape) * 3e5   # beyond the 32-bit walk
    pts[2::1009] = np.nan
    return blob.astype(np.float32), t, (pts - t).astype(np.float32)


@pytest.mark.parametrize("dims,batch", [((37, 23, 11), 0), ((1, 9, 700), 0), ((700, 8, 3), 0), ((131, 97, 70), 16),
                                        ((403, 398, 201), 0), ((700, 690, 330), 0), ((1030, 1200, 1100), 0)])
@pytest.mark.parametrize("bricks", [False, True])
def test_forms_equal_the_oracle(dims, batch, bricks):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(sum(dims))
    n = _bricks_from(dims) - (0 if bricks else 1)
    if batch and bricks:
        n = max(n, 3 * (1 << batch) + 17)   # a batch of 2^16 is the smallest
    s = 0.01
    blob, t, pts = _scene(rng, dims, s, n)
    note(f"clearing forms {dims} n={n}")
    m, om = vm.Map((0.0, 0.0, 0.0), s, dims, 18, insert_batch_log2=batch), oracle.OracleMap((0.0, 0.0, 0.0), s, dims)
    for step in range(2):
        m.insert(torch.from_numpy(blob).cuda())
        om.insert(blob)
        m.clear_rays(torch.from_numpy(pts).cuda(), None, t)
        om.clear_rays(pts, np.eye(3), t)
        assert_map_equal(m, om)
        # and the other form after it
        few = pts[: 1000 + step]
        m.insert(torch.from_numpy(blob[::2].copy()).cuda())
        om.insert(blob[::2])
        m.clear_rays(torch.from_numpy(few).cuda(), None, t)
        om.clear_rays(few, np.eye(3), t)
        assert_map_equal(m, om)
    m.close()


@pytest.mark.parametrize("many_first", [False, True])
def test_many_rays_captured(many_first):
    import torch
    import paper_2510_01592_amd as vm
    dims, s = (160, 150, 90), 0.01
    rng = np.random.default_rng(3)
    n = _bricks_from(dims) + 100
    blob, t, pts = _scene(rng, dims, s, n)
    m, om = vm.Map((0.0, 0.0, 0.0), s, dims, 18), oracle.OracleMap((0.0, 0.0, 0.0), s, dims)
    db, dp = torch.from_numpy(blob).cuda(), torch.from_numpy(pts).cuda()
    first = pts if many_first else pts[:50]
    m.clear_rays(torch.from_numpy(first).cuda(), None, t)   # (the map is empty)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    note(f"clearing captured, many rays first: {many_first}")
    with torch.cuda.stream(st), vm.capture(st) as cap:
        m.insert(db, stream=st)
        m.clear_rays(dp, None, t, stream=st)
    for _ in range(3):
        cap.graph.launch(st)
        torch.cuda.synchronize()
        om.insert(blob)
        om.clear_rays(pts, np.eye(3), t)
        assert_map_equal(m, om)
    m.close()


def test_few_rays_take_two_bitmaps():
    import torch
    import paper_2510_01592_amd as vm
    dims = (2100, 2100, 60)
    m = vm.Map((0.0, 0.0, 0.0), 0.01, dims, 12)
    p = torch.rand((1000, 3), device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    m.clear_rays(p, None, (10.0, 10.0, 0.3))
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    assert used <= 2 * int(np.prod(dims)) // 8 + (8 << 20), used   # (and what the allocator rounds up)
    m.close()
