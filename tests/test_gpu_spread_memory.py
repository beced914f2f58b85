"""Spread queries without the memory for their order: the call answers in the given order."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev
from test_gpu_query_spread import _mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("hinted", [False, True])
def test_no_memory_for_the_order(device, hinted, monkeypatch):
    import paper_2606_00444_amd as mg
    from paper_2606_00444_amd import api
    V, F = _mesh(False, device)
    bvh = mg.lbvh_build(V, F)
    Q = dev(np.random.default_rng(1).uniform(-1.5, 1.5, size=(3, 3000)).astype(np.float32), device)
    hint = torch.randint(0, F.shape[1], (3000,), dtype=torch.int32, device=device) if hinted else None
    ref = mg.closest_point_query(bvh, V, Q, hint=hint)
    out = api._query_out(3000, device, True, True, True, False)
    tried = []

    def empty(*a, **kw):
        tried.append(a)
        raise torch.OutOfMemoryError("no memory")
    monkeypatch.setattr(api, "_SPREAD_COLD", (0, 1))
    monkeypatch.setattr(api, "_SPREAD_HINTED", (0, 1))
    monkeypatch.setattr(torch, "empty", empty)
    mg.closest_point_query(bvh, V, Q, hint=hint, out=out)
    monkeypatch.undo()
    assert len(tried) == 1
    for key in ("face", "point", "bary", "dist2"):
        assert torch.equal(out[key], ref[key]), key
