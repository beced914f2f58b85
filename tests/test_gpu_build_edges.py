"""The build at the sizes and key distributions where its kernels change form: workgroup
and search-window edges of the hierarchy, every tile shape of the sort, and skewed codes
(few long ranges, or all of them), bitwise against the oracle's tree."""

import ctypes

import numpy as np
import pytest

from gpu_helpers import need_gpu, dev
from paper_2606_00444_amd._lib import LbvhHeader
from test_gpu_lbvh import _check_build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


def _points(dist, n, rng):
    if dist == "uniform":
        P = rng.uniform(-1, 1, size=(3, n))
    elif dist == "same":                       # one code: the tree follows the indices
        P = np.full((3, n), 0.25)
    else:                                      # one far point squeezes the others into a few codes
        P = 1e-3 * rng.normal(size=(3, n))
        P[:, n // 2] = 50.0
    return P.astype(np.float32)


@pytest.mark.parametrize("dist", ["uniform", "same", "outlier"])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 66, 129, 255, 256, 257, 258, 320, 511, 513, 1025, 5000])
def test_build_window_edges(device, n, dist):
    import paper_2606_00444_amd as mg
    P = _points(dist, n, np.random.default_rng(n))
    _check_build(mg.lbvh_build(dev(P, device), None), P, None)


@pytest.mark.parametrize("dist", ["uniform", "outlier"])
@pytest.mark.parametrize("n", [131072, 131073, 262145, 524289])
def test_build_sort_tiles(device, n, dist):
    """512-, 1024-, 2048- and 4096-key tiles, the last one nearly empty."""
    import paper_2606_00444_amd as mg
    P = _points(dist, n, np.random.default_rng(n))
    print(f"build: {n} points, {dist}", flush=True)
    _check_build(mg.lbvh_build(dev(P, device), None), P, None)


@pytest.mark.parametrize("faces", [False, True])
@pytest.mark.parametrize("dist", ["uniform", "same", "outlier"])
@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
def test_build_one_workgroup_sort(device, n, dist, faces):
    """One workgroup's sort of 1, 2 and 4 keys a thread, full and one off, and the first
    size of the tiled sort."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(n)
    P = _points(dist, n + 2 if faces else n, rng)
    F = np.stack([np.arange(n), np.arange(n) + 1, np.arange(n) + 2]).astype(np.int32) if faces else None
    _check_build(mg.lbvh_build(dev(P, device), None if F is None else dev(F, device)), P, F)


@pytest.mark.parametrize("n,faces", [(524289, True), (1400000, False)])
def test_refit_of_2048_leaf_subtrees(device, n, faces):
    """1024-thread workgroups, with up to 1024 top nodes (one a thread) and more (two)."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(n)
    P = (rng.normal(size=(3, n + 2 if faces else n)) ** 3).astype(np.float32)
    F = np.stack([np.arange(n), np.arange(n) + 1, np.arange(n) + 2]).astype(np.int32) if faces else None
    print(f"refit: {n}, faces {faces}", flush=True)
    Pd = dev(P, device)
    bvh = mg.lbvh_build(Pd, None if F is None else dev(F, device))
    mg.lbvh_refit(bvh, Pd)
    _check_build(bvh, P, F)
    hdr = LbvhHeader.from_buffer_copy(bvh.buf[:ctypes.sizeof(LbvhHeader)].cpu().numpy().tobytes())
    assert (hdr.n_top > 1024) == (n > 1000000)
