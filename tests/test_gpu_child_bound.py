"""The traversals against the all-faces kernel where their lower bounds, batches and
k-nearest lists can go wrong: meshes far from the origin and at extreme scales (the
rounding margins of the slab and ball bound), needle and flat boxes, face and query
counts at the edges of the batches, and lists longer than the mesh."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev, check_knn_result
from synth.meshes import icosphere, uv_sphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


def _mesh(shape, scale, offset, rng):
    v, f = uv_sphere(24, 17) if shape != "needle" else icosphere(3)
    v = v + 0.02 * rng.normal(size=v.shape)
    v = v * {"ball": (1, 1, 1), "flat": (1, 1, 1e-4), "needle": (1, 1e-3, 1e-3)}[shape]
    V = (scale * (v + offset)).astype(np.float32).T
    lo, hi = V.min(1, keepdims=True), V.max(1, keepdims=True)
    mid = 0.5 * (lo + hi)
    near = V[:, ::7] + (1e-3 * (hi - lo)) * rng.normal(size=(3, V[:, ::7].shape[1]))
    Q = np.concatenate([mid + 1e-3 * (hi - lo) * rng.normal(size=(3, 40)),        # nearly equidistant from many faces
                        rng.uniform(lo - (hi - lo), hi + (hi - lo), size=(3, 400)), near], axis=1)
    return np.ascontiguousarray(V), np.ascontiguousarray(f.T.astype(np.int32)), Q.astype(np.float32)


@pytest.mark.parametrize("shape", ["ball", "flat", "needle"])
@pytest.mark.parametrize("scale,offset", [(1.0, 0.0), (1.0, 200.0), (1e-6, 3.0), (1e6, 0.0), (1.0, 5000.0)])
def test_traversals_match_all_faces(device, shape, scale, offset):
    """Faces equal, distances bitwise: the bound may never drop a face that the all-faces
    kernel finds nearest (ties of the float32 distance to the lowest id in both)."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(7)
    V, F, Q = (dev(x, device) for x in _mesh(shape, scale, offset, rng))
    ref = mg.closest_point_bruteforce(V, F, Q, normal=True)
    bvh = mg.lbvh_build(V, F)
    for kw in ({}, {"kernel": "lane"}, {"kernel": "batch", "batch": 16, "seed": True},
               {"kernel": "batch", "batch": 32, "seed": True}, {"kernel": "batch", "batch": 16},
               {"hint": ref["face"].roll(1)}, {"hint": ref["face"]}):
        r = mg.closest_point_query(bvh, V, Q, normal=True, **kw)
        assert torch.equal(r["dist2"], ref["dist2"]), kw
        assert torch.equal(r["face"], ref["face"]), kw
        for key in ("point", "bary", "normal"):
            assert torch.equal(r[key], ref[key]), (kw, key)


@pytest.mark.parametrize("nf", [1, 2, 3, 7, 9, 64, 65])
@pytest.mark.parametrize("k", [2, 3, 5, 8])
def test_knn_small_meshes_and_ragged_counts(device, nf, k):
    """Fewer faces than places, one to two wave-fulls of faces, 1 to 70 queries."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(100 * nf + k)
    c = rng.uniform(-1, 1, size=(nf, 1, 3))
    V = (c + 0.2 * rng.normal(size=(nf, 3, 3))).reshape(-1, 3).T.astype(np.float32)
    F = np.arange(3 * nf, dtype=np.int32).reshape(nf, 3).T.copy()
    Vd, Fd = dev(np.ascontiguousarray(V), device), dev(F, device)
    bvh = mg.lbvh_build(Vd, Fd)
    for nq in (1, 5, 70):
        Q = rng.uniform(-1.5, 1.5, size=(3, nq)).astype(np.float32)
        r = mg.knn_surface_query(bvh, Vd, dev(Q, device), k=k, eps=1e-6)
        check_knn_result(r, V, F, Q, k, 1e-6, float("inf"))


@pytest.mark.parametrize("k", [1, 2, 4, 8])
def test_knn_does_not_depend_on_the_batch(device, k):
    """The queries per wave follow the query count: the same queries alone and among 33,000."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(5)
    V, F, _ = _mesh("ball", 1.0, 0.0, rng)
    Q = rng.uniform(-1.2, 1.2, size=(3, 33000)).astype(np.float32)
    Vd, Fd, Qd = dev(V, device), dev(F, device), dev(Q, device)
    bvh = mg.lbvh_build(Vd, Fd)
    whole = mg.knn_surface_query(bvh, Vd, Qd, k=k, eps=1e-6, max_dist2=0.3)
    for n in (333, 4100, 8200, 16400):
        part = mg.knn_surface_query(bvh, Vd, Qd[:, :n].contiguous(), k=k, eps=1e-6, max_dist2=0.3)
        for key in ("face", "dist2", "point"):
            assert torch.equal(part[key], whole[key][:, :n]), (n, key)


@pytest.mark.parametrize("nf", [2, 300, 5000])
@pytest.mark.parametrize("kind", ["doubling", "same"])
def test_cold_queries_on_deep_trees(device, nf, kind):
    """A seed descent that passes by more than the stack holds starts from the root again:
    sizes doubling from face to face, then coincident faces, both far deeper than a mesh."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(nf)
    if kind == "doubling":
        c = np.exp2(-(np.arange(nf) % 24)).reshape(nf, 1, 1) * np.ones((1, 1, 3))
        V = c * (1 + 0.2 * rng.normal(size=(nf, 3, 3)))
    else:
        V = np.broadcast_to(rng.normal(size=(1, 3, 3)), (nf, 3, 3)) + np.zeros((nf, 1, 1))
        V = np.concatenate([V, 5 + rng.normal(size=(3, 3, 3))])
    V = np.ascontiguousarray(V.reshape(-1, 3).T.astype(np.float32))
    F = np.ascontiguousarray(np.arange(V.shape[1], dtype=np.int32).reshape(-1, 3).T)
    Q = np.concatenate([np.exp2(rng.uniform(-24, 1, size=(1, 500))) * rng.uniform(0.9, 1.1, size=(3, 500)),
                        rng.uniform(-1, 6, size=(3, 500))], axis=1).astype(np.float32)
    Vd, Fd, Qd = dev(V, device), dev(F, device), dev(Q, device)
    ref = mg.closest_point_bruteforce(Vd, Fd, Qd)
    bvh = mg.lbvh_build(Vd, Fd)
    for batch in (1, 2, 4, 8, 16, 32):
        r = mg.closest_point_query(bvh, Vd, Qd, kernel="batch", batch=batch, seed=True)
        assert torch.equal(r["face"], ref["face"]) and torch.equal(r["dist2"], ref["dist2"]), batch
    if kind == "doubling":
        for k in (2, 4):
            check_knn_result(mg.knn_surface_query(bvh, Vd, Qd, k=k, eps=1e-6), V, F, Q, k, 1e-6, float("inf"))


@pytest.mark.parametrize("n", [2, 63, 65, 255, 256, 257, 1279, 1280])
@pytest.mark.parametrize("max_dist2", [float("inf"), 0.02])
def test_scan_matches_all_faces(device, n, max_dist2):
    """Every leaf scanned, in groups of 64 and fours of them: one, a full set and a remainder;
    ties of coincident faces, points that are no numbers or overflow, hints of no use."""
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(n)
    V = (rng.uniform(-1, 1, size=(n, 1, 3)) + 0.2 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    V[n // 2:n // 2 + 9] = V[0]                               # faces in one place
    V = np.ascontiguousarray(V.reshape(-1, 3).T)
    F = np.arange(3 * n, dtype=np.int32).reshape(n, 3).T.copy()
    Q = rng.uniform(-1.5, 1.5, size=(3, 301)).astype(np.float32)
    Q[:, 0], Q[:, 1], Q[:, 2], Q[0, 3] = np.nan, 1e25, V[:, 0], np.inf
    Vd, Fd, Qd = dev(V, device), dev(F, device), dev(Q, device)
    bvh = mg.lbvh_build(Vd, Fd)
    walk = mg.closest_point_query(bvh, Vd, Qd, max_dist2, normal=True, kernel="batch", batch=4)
    ref = mg.closest_point_bruteforce(Vd, Fd, Qd, max_dist2, normal=True)
    hint = torch.randint(-1, n + 1, (301,), dtype=torch.int32, device=device)
    for h in (None, hint):
        r = mg.closest_point_query(bvh, Vd, Qd, max_dist2, normal=True, hint=h)
        for key in r:
            assert torch.equal(r[key].nan_to_num(7.0), walk[key].nan_to_num(7.0)), key
            assert torch.equal(r[key][..., 4:], ref[key][..., 4:]), key
    P = np.ascontiguousarray(V[:, ::3])
    pts = mg.lbvh_build(dev(P, device))
    i, d = mg.nearest_point_query(pts, dev(P, device), Qd, max_dist2)
    j, e = mg.nearest_point_query(pts, dev(P, device), Qd, max_dist2, kernel="batch", batch=4)
    assert torch.equal(i, j) and torch.equal(d, e)


@pytest.mark.parametrize("faces,n,nq", [(True, 1280, 4096), (True, 1281, 4096), (True, 1280, 4097),
                                        (False, 3072, 4096), (False, 3073, 4096), (False, 3072, 4097)])
def test_scan_rule_edges(device, faces, n, nq):
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(n + nq)
    P = dev(rng.uniform(-1, 1, size=(3, n + 2 if faces else n)).astype(np.float32), device)
    Q = dev(rng.uniform(-1.2, 1.2, size=(3, nq)).astype(np.float32), device)
    if faces:
        F = dev(np.stack([np.arange(n) + s for s in range(3)]).astype(np.int32), device)
        bvh = mg.lbvh_build(P, F)
        r = mg.closest_point_query(bvh, P, Q, normal=True)
        w = mg.closest_point_query(bvh, P, Q, normal=True, kernel="batch", batch=4)
        assert all(torch.equal(r[key], w[key]) for key in r)
    else:
        bvh = mg.lbvh_build(P)
        r, w = mg.nearest_point_query(bvh, P, Q), mg.nearest_point_query(bvh, P, Q, kernel="batch", batch=4)
        assert torch.equal(r[0], w[0]) and torch.equal(r[1], w[1])
