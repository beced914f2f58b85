"""Batches without the seed descent: they search no more of the tree than with it, and
queries out of max_dist2 at the root still cost nothing."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev
from synth.meshes import uv_sphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("batch", [1, 4, 16, 32])
def test_unseeded_batches_search_no_more(device, batch):
    """The same queries with and without `seed`: results bitwise equal, and as many node
    expansions (which only the order of the rounds may change a little)."""
    import paper_2606_00444_amd as mg
    v, f = uv_sphere(100, 51)
    V, F = dev(np.ascontiguousarray(v.T.astype(np.float32)), device), dev(np.ascontiguousarray(f.T.astype(np.int32)), device)
    Q = dev(np.random.default_rng(2).uniform(-1.2, 1.2, size=(3, 4097)).astype(np.float32), device)
    bvh = mg.lbvh_build(V, F)
    res, counts = [], []
    for seed in (True, False):
        c = torch.zeros(4, dtype=torch.int64, device=device)
        res.append(mg.closest_point_query(bvh, V, Q, kernel="batch", batch=batch, seed=seed, counters=c))
        counts.append(c.cpu().tolist())
    for key in ("face", "point", "bary", "dist2"):
        assert torch.equal(res[0][key], res[1][key]), key
    assert counts[1][0] <= 1.05 * counts[0][0], counts
    ref = mg.closest_point_bruteforce(V, F, Q)
    assert torch.equal(res[1]["face"], ref["face"])


def test_queries_out_of_reach_expand_nothing(device):
    import paper_2606_00444_amd as mg
    v, f = uv_sphere(100, 51)
    V, F = dev(np.ascontiguousarray(v.T.astype(np.float32)), device), dev(np.ascontiguousarray(f.T.astype(np.int32)), device)
    Q = dev(np.random.default_rng(3).uniform(3, 4, size=(3, 1000)).astype(np.float32), device)
    bvh = mg.lbvh_build(V, F)
    c = torch.zeros(4, dtype=torch.int64, device=device)
    r = mg.closest_point_query(bvh, V, Q, 0.01, kernel="batch", batch=8, seed=False, counters=c)
    assert (r["face"] == -1).all() and c.cpu().tolist() == [0, 0, 0, 1000]


@pytest.mark.parametrize("batch", [1, 8, 32])
def test_unseeded_point_batches_search_no_more(device, batch):
    import paper_2606_00444_amd as mg
    g = torch.Generator(device=device).manual_seed(6)
    P = torch.rand(3, 20000, device=device, generator=g)
    Q = torch.rand(3, 3000, device=device, generator=g)
    bvh = mg.lbvh_build(P)
    res, counts = [], []
    for seed in (True, False):
        c = torch.zeros(4, dtype=torch.int64, device=device)
        res.append(mg.nearest_point_query(bvh, P, Q, kernel="batch", batch=batch, seed=seed, counters=c))
        counts.append(c.cpu().tolist())
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    assert counts[1][0] <= 1.05 * counts[0][0], counts
