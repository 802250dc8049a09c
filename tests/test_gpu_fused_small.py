"""The persistent pass where its smallest clusters (fewer than 256 points) are
taken in turn instead of from the queue: none, only and some of them, one
workgroup's worth and many times that, beside clusters at the line and empty
ones -- planes, inliers and polygons the same bits as the two-pass calls', for
splits with one and with several chunks."""
import numpy as np
import pytest

from tests.gpu_util import bits, cluster_tensors, hulls_np, note, planes_np, run_planes_and_hulls

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(255,), (256,), (255, 256, 257, 0, 1), (5000, 256), "tiny", "mixed"])
@pytest.mark.parametrize("cfg", [None, dict(hyp_chunk=64, small_max=0, groups_per_cu=1), dict(hyp_chunk=128, small_max=256)])
def test_equal_to_two_passes(sizes, cfg):
    import torch
    import paper_2510_01592_amd as vm
    rng = np.random.default_rng(5)
    if sizes == "tiny":
        sizes = rng.integers(0, 40, 9000)
    elif sizes == "mixed":
        sizes = np.r_[rng.integers(0, 300, 3000), rng.integers(250, 260, 50), rng.integers(4000, 13_000, 20)]
        rng.shuffle(sizes)
    off = np.zeros(len(sizes) + 1, np.uint32)
    off[1:] = np.cumsum(sizes)
    xyz = (rng.random((int(off[-1]), 3)) * [1.0, 0.7, 0.02]).astype(np.float32)
    tag = np.arange(len(sizes), dtype=np.uint32) * 3 + 1
    K, N, H = len(tag), len(xyz), 130
    T = cluster_tensors(off, xyz, tag)
    cl = vm.cluster_view(T["off"], T["x"], T["y"], T["z"], T["tag"], T["meta"])
    pb, hb = run_planes_and_hulls(vm, cl, K, N, H, 0.01, 7, 2)
    ref, refh = planes_np(pb), hulls_np(hb)
    vm.set_fused_config(None)
    if cfg:
        vm.set_fused_config(cfg)
    note(f"persistent, {K} clusters, {cfg}")
    work = torch.empty(vm.workspace_bytes(K, N, H), dtype=torch.uint8, device="cuda")
    p, h = vm.PlaneBuffers.alloc(K, N, H, with_all=True), vm.HullBuffers.alloc(K, N)
    vm.planes_hulls(cl, vm.ransac_params(H, 0.01, 7, 2), p, h, work)
    torch.cuda.synchronize()
    vm.set_fused_config(None)
    P, Hh = planes_np(p), hulls_np(h)
    n, v = int(ref["in_off"][K]), int(refh["v_off"][K])
    for k in ("best", "nin", "in_off", "counts", "status"):
        assert np.array_equal(P[k], ref[k]), k
    for k in ("plane", "hyp"):
        assert np.array_equal(bits(P[k]), bits(ref[k])), k
    assert np.array_equal(P["in_idx"][:n], ref["in_idx"][:n])
    assert np.array_equal(Hh["v_off"], refh["v_off"]) and np.array_equal(Hh["v_idx"][:v], refh["v_idx"][:v])
    assert np.array_equal(bits(Hh["v_xyz"][:v]), bits(refh["v_xyz"][:v])) and np.array_equal(Hh["area"], refh["area"])
