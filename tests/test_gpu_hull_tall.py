"""Polygons of clusters that reach much further along the plane's normal than in
the plane, and of coordinates up to the largest floats: caller-given oblique
planes and inlier lists, widths of 4e-5 to 1e30 m, straight-edged outlines with
many vertices -- vertex lists and projected vertices exact, areas within 1e-5,
against the oracle.  (With W the spread along the normal and S the width, the
fp64 projections both sides start from err by about 1e-16 W, which for W = 1e5 S
is 1e-11 S: far below the outlines' turns of 1e-3 S.)"""
import numpy as np
import pytest

import oracle
from tests.gpu_util import bits, cluster_tensors, hulls_np, note

pytestmark = pytest.mark.gpu


def _outline(rng, n, width):
    """points on and inside a rounded square: four edges that bulge by 1 %, every edge point a vertex"""
    t = rng.uniform(-1, 1, n)
    edge = np.c_[t, 1.0 + 0.01 * (1 - t * t)]
    q = rng.integers(0, 4, n)
    c, s = np.cos(q * np.pi / 2), np.sin(q * np.pi / 2)
    p = np.c_[c * edge[:, 0] - s * edge[:, 1], s * edge[:, 0] + c * edge[:, 1]]
    inner = rng.random(n) < 0.8
    p[inner] *= 0.9 * rng.random((inner.sum(), 1))
    return p * width / 2


@pytest.mark.parametrize("ratio", [1.0, 1e3, 1e4, 1e5])
@pytest.mark.parametrize("width", [4e-5, 1.0, 1e30])
def test_hulls_of_tall_clusters_equal_the_oracle(ratio, width):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(int(ratio) + 5)
    parts, planes = [], []
    for n in (65, 700, 1500, 4000, 4000, 4000, 4000, 4000):
        nrm = rng.normal(size=3)
        nrm /= np.linalg.norm(nrm)
        a = np.cross(nrm, [1.0, 0.0, 0.0])
        a /= np.linalg.norm(a)
        b = np.cross(nrm, a)
        uv = _outline(rng, n, width)
        h = rng.uniform(-0.5, 0.5, n) * width * ratio
        parts.append((uv[:, :1] * a + uv[:, 1:] * b + h[:, None] * nrm).astype(np.float32))
        planes.append(np.r_[nrm, 0.0].astype(np.float32))
    off = np.zeros(len(parts) + 1, np.uint32)
    off[1:] = np.cumsum([len(p) for p in parts])
    xyz, tag = np.concatenate(parts), np.arange(len(parts), dtype=np.uint32)
    K, N = len(tag), len(xyz)
    T = cluster_tensors(off, xyz, tag)
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    pb, hb = vm.PlaneBuffers.alloc(K, N, 1), vm.HullBuffers.alloc(K, N)
    pb.plane.copy_(torch.from_numpy(np.stack(planes)))
    pb.in_off.copy_(T["off"])
    pb.in_idx.copy_(torch.from_numpy(np.concatenate([np.arange(len(p)) for p in parts]).astype(np.int32)))
    work = torch.empty(vm.workspace_bytes(K, N, 1), dtype=torch.uint8, device="cuda")
    note(f"tall clusters ratio {ratio:g} width {width:g}")
    vm.hulls(cl, pb, hb, work)
    torch.cuda.synchronize()
    H = hulls_np(hb)
    for k, p in enumerate(parts):
        ref = oracle.hull(p[:, 0], p[:, 1], p[:, 2], planes[k])
        va, vb = int(H["v_off"][k]), int(H["v_off"][k + 1])
        assert np.array_equal(H["v_idx"][va:vb], ref.idx), (k, vb - va, len(ref.idx))
        assert np.array_equal(bits(H["v_xyz"][va:vb]), bits(ref.xyz)), k
        assert abs(H["area"][k] - ref.area) <= 1e-5 * abs(ref.area), k
