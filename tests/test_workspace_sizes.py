"""The sizes of the caller's workspaces and the largest calls the allocation-free
form takes: a buffer of a remembered size stays large enough, and the same calls
are accepted, whatever the arrays inside are used for (no GPU needed)."""
import ctypes

import pytest

import paper_2510_01592_amd as vm


def _sum(*sizes):
    return sum((s + 255) & ~255 for s in sizes)


def _two_pass(k, n, h):
    kh, ht, nt = k * h, n // 1024 + k + 2, n // 4096 + k + 2
    blk = (n + k + 2 + 4095) // 4096 + 128
    return _sum(4 * kh, 16 * kh, 4 * (k + 2), 4 * nt, 4 * (k + 2), 4 * nt, 4 * (n + 1), 4 * blk, 4 * (k + 2), 4 * (k + 2),
                4 * (n + k + 2), 8 * (n + 1), 8 * (n + 1), 4 * (n + 1), 4 * (k + 2), 64 * ht, 32 * ht, 144 * k + 8,
                4 * (k + 1), 4 * (k + 1), 256)


def _persistent(k, n, h):
    return _sum((n // 4096 + k + 1) * h * 4, 16 * k * h, *([4 * (k + 1)] * 8), 4 * (n + 1), 4 * (n + k + 2), 8 * (n + 1),
                8 * (n + 1), 4 * (n + 1), 256)


def _merged(k, n, h):
    kc, nc = k + 1, n + 1
    return _two_pass(k, n, h) + _sum(64, 4 * kc, 4 * kc, 4 * kc, 4 * nc, 4 * nc, 4 * nc, 64, 16 * kc, 4 * kc, 4 * kc, 8 * kc,
                                     4 * k * h, 16 * k * h, 4 * kc, 4 * nc, 4 * kc, 4 * nc, 12 * nc, 4 * kc, 256)


SHAPES = [(1, 1, 1), (1, 2_388_319, 1), (3, 0, 5), (7, 100, 64), (63, 4095, 65), (64, 4096, 256), (100, 64, 1024),
          (2000, 50_000_000, 1024), (65_536, 1000, 16), (65_536, 1 << 21, 512), (70_001, 1 << 20, 3)]


@pytest.mark.parametrize("k,n,h", SHAPES)
def test_sizes(k, n, h):
    assert vm.workspace_bytes(k, n, h) == max(_two_pass(k, n, h), _persistent(k, n, h))
    assert vm.multi_workspace_bytes(k, n, h) == _merged(k, n, h)


@pytest.mark.parametrize("k,n,h", [(1, 2_388_319, 1), (2000, 2_003_999, 256)])
def test_largest_calls_of_the_allocation_free_form(k, n, h):
    import torch
    if torch.cuda.is_available():
        pytest.skip("the pointers below are none of a GPU's")
    assert _two_pass(k, n, h) <= vm.NOALLOC_WORK_BYTES < _two_pass(k, n + 1, h)

    def call(points):
        cl = vm.Clusters(k, points, 8, 8, 8, 8, 8, None, 8)
        pl = vm.Planes(k, 1, 8, 8, 8, 8, 8, None, None, 8)
        return vm.lib().vm_ransac_planes_noalloc(ctypes.byref(cl), ctypes.byref(vm.RansacParams(h, 0.01, 1, 0, 0)),
                                                 ctypes.byref(pl), None)
    assert call(n + 1) == vm.VM_E_CAPACITY
    assert call(n) == vm.VM_E_DEVICE   # past the checks: there is no device here
