"""Batches whose queries start in different ways: some from a hinted face, whose roots go
on top of what the other queries' seed descents kept."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


def _deep(nf, rng):
    """Faces whose sizes halve from one to the next, 24 times over, and as many coincident
    ones at the small end: far deeper than a mesh."""
    c = np.exp2(-(np.arange(nf) % 24)).reshape(nf, 1, 1)
    V = c * (1 + 0.2 * rng.normal(size=(nf, 3, 3)))
    V[nf // 2:] = V[23]
    V = np.ascontiguousarray(V.reshape(-1, 3).T.astype(np.float32))
    return V, np.ascontiguousarray(np.arange(3 * nf, dtype=np.int32).reshape(nf, 3).T)


@pytest.mark.parametrize("nf", [60, 2000])
@pytest.mark.parametrize("batch", [2, 8, 16])
@pytest.mark.parametrize("hinted", [1, 5, 15])
def test_hinted_and_cold_queries_in_one_batch(device, nf, batch, hinted):
    """`hinted` of every 16 queries have a face to start from."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(nf + batch)
    V, F = _deep(nf, rng)
    Q = (np.exp2(rng.uniform(-24, 1, size=(1, 1000))) * rng.uniform(0.9, 1.1, size=(3, 1000))).astype(np.float32)
    Vd, Fd, Qd = dev(V, device), dev(F, device), dev(Q, device)
    ref = mg.closest_point_bruteforce(Vd, Fd, Qd)
    bvh = mg.lbvh_build(Vd, Fd)
    hint = torch.randint(0, nf, (1000,), dtype=torch.int32, device=device)
    hint[torch.arange(1000, device=device) % 16 >= hinted] = -1
    r = mg.closest_point_query(bvh, Vd, Qd, kernel="batch", batch=batch, seed=True, hint=hint)
    assert torch.equal(r["face"], ref["face"]) and torch.equal(r["dist2"], ref["dist2"])
    assert int(bvh.buf[:16].view(torch.int32)[2]) == 0           # the header's error word
