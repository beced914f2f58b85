"""The index SDF's update with face records at the node counts from which it takes them."""

import ctypes

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("k,least", [(1, 13 << 16), (2, 1 << 18), (4, 1 << 17), (8, 1 << 16)])
def test_records_change_nothing_at_the_rule(device, k, least):
    """Just below and just above (grids of 1,023 nodes a layer, no whole number of
    workgroups): the values and faces of the plain update, ids outside the mesh ignored, and
    the records written above only."""
    from paper_2606_00444_amd import _lib, sdf
    from paper_2606_00444_amd.api import _ptr, _stream
    rng = np.random.default_rng(k)
    nv, nf = 2301, 4099
    V = dev(rng.normal(size=(3, nv)).astype(np.float32), device)
    F = dev(rng.integers(0, nv, size=(3, nf)).astype(np.int32), device)
    lib = _lib.load()
    for above in (False, True):
        dims = (31, 33, least // 1023 + above)
        n = dims[0] * dims[1] * dims[2]
        assert sdf.records_bytes(nf, k, dims) == (48 * nf if above else 0)
        face_k = torch.randint(-1, nf + 1, (k, n), dtype=torch.int32, device=device)
        rec = torch.full((12 * nf,), 7.0, device=device)
        out = []
        for records, size in ((None, 0), (_ptr(rec), 48 * nf)):
            d, w = torch.empty(n, device=device), torch.empty(n, dtype=torch.int32, device=device)
            assert lib.mg_sdf_update_records(_ptr(V), nv, _ptr(F), nf, _ptr(face_k), k, -1.0, -1.0, -1.0, 0.05, *dims,
                                             _ptr(d), _ptr(w), records, ctypes.c_size_t(size), _stream()) == 0
            out.append((d, w))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
        assert bool((rec != 7.0).any()) == above
