"""The batch kernel by name on meshes so small that the automatic choice scans them: its
hinted starts far from the origin, at extreme scales and in flat and needle boxes, and
queries that are no numbers or overflow through the seed descent."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev
from test_gpu_child_bound import _mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("shape", ["ball", "flat", "needle"])
@pytest.mark.parametrize("scale,offset", [(1.0, 0.0), (1.0, 200.0), (1e-6, 3.0), (1e6, 0.0), (1.0, 5000.0)])
@pytest.mark.parametrize("batch", [1, 4, 16, 32])
def test_hinted_batches_match_all_faces(device, shape, scale, offset, batch):
    import paper_2606_00444_amd as mg
    V, F, Q = (dev(x, device) for x in _mesh(shape, scale, offset, np.random.default_rng(7)))
    ref = mg.closest_point_bruteforce(V, F, Q, normal=True)
    bvh = mg.lbvh_build(V, F)
    some = ref["face"].roll(1)
    some[::3] = -1                                    # these walk down, if the seed is on
    for hint in (ref["face"], ref["face"].roll(1), some):
        for seed in (False, True):
            r = mg.closest_point_query(bvh, V, Q, normal=True, kernel="batch", batch=batch, seed=seed, hint=hint)
            for key in ref:
                assert torch.equal(r[key], ref[key]), (seed, key)


@pytest.mark.parametrize("nf", [300, 5000])
@pytest.mark.parametrize("batch", [1, 4, 16, 32])
@pytest.mark.parametrize("max_dist2", [float("inf"), 0.02])
def test_queries_that_are_no_numbers(device, nf, batch, max_dist2):
    """They end as by the walk from the root, with no face if they are not numbers, and
    leave the other queries of their batch alone."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(nf)
    V = (rng.uniform(-1, 1, size=(nf, 1, 3)) + 0.2 * rng.normal(size=(nf, 3, 3))).astype(np.float32)
    V = np.ascontiguousarray(V.reshape(-1, 3).T)
    F = np.arange(3 * nf, dtype=np.int32).reshape(nf, 3).T.copy()
    Q = rng.uniform(-1.5, 1.5, size=(3, 301)).astype(np.float32)
    odd = np.arange(0, 300, 5)
    Q[rng.integers(0, 3, size=odd.size), odd] = np.resize(np.array([np.nan, np.inf, -np.inf, 1e25], np.float32), odd.size)
    fine = np.setdiff1d(np.arange(301), odd)
    Vd, Fd, Qd = dev(V, device), dev(F, device), dev(Q, device)
    bvh = mg.lbvh_build(Vd, Fd)
    ref = mg.closest_point_bruteforce(Vd, Fd, Qd, max_dist2, normal=True)
    r = mg.closest_point_query(bvh, Vd, Qd, max_dist2, normal=True, kernel="batch", batch=batch, seed=True)
    walk = mg.closest_point_query(bvh, Vd, Qd, max_dist2, normal=True, kernel="batch", batch=4)
    for key in ref:
        assert torch.equal(r[key][..., fine], ref[key][..., fine]), key
        assert torch.equal(r[key].nan_to_num(7.0), walk[key].nan_to_num(7.0)), key
    assert (r["face"][torch.from_numpy(np.isnan(Q).any(0)).to(device)] == -1).all()
    k = mg.knn_surface_query(bvh, Vd, Qd, k=3, eps=1e-6, max_dist2=max_dist2)
    alone = mg.knn_surface_query(bvh, Vd, Qd[:, fine].contiguous(), k=3, eps=1e-6, max_dist2=max_dist2)
    for key in alone:
        assert torch.equal(k[key][..., fine], alone[key]), key
    assert (k["face"][:, torch.from_numpy(np.isnan(Q).any(0)).to(device)] == -1).all()
