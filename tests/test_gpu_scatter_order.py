"""Scatters in a processing order, and the reductions' one-workgroup and two-array forms.

Inputs are small integers and weights multiples of 1/4, so every product and partial sum is
exact in float32 (and float64): results are compared bitwise whatever the order of the adds."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 20000])
def test_point_mesh_backward_in_any_order(device, n):
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(n)
    nv, nf = 40, 60
    V = rng.integers(-4, 5, size=(3, nv)).astype(np.float32)
    F = rng.integers(0, nv, size=(3, nf)).astype(np.int32)
    Y, C = (rng.integers(-4, 5, size=(3, n)).astype(np.float32) for _ in range(2))
    face = rng.integers(-1, nf, size=n).astype(np.int32)
    w = np.array([[0, 0], [0.25, 0.5], [1, 0], [0.5, 0.5]], np.float32)[rng.integers(0, 4, size=n)].T.copy()
    want = np.zeros((3, nv))
    full = np.concatenate([1 - w.sum(0, keepdims=True), w])
    ok = face >= 0
    for k in range(3):
        for c in range(3):
            np.add.at(want[c], F[k, face[ok]], (-2.0 * full[k] * (Y - C)[c])[ok])
    rec = {"face": dev(face, device), "point": dev(C, device), "bary": dev(w, device)}
    args = (dev(V, device), dev(F, device), dev(Y, device), rec, 1.0)
    by_face = np.argsort(face, kind="stable").astype(np.int32)          # long runs
    for order in (None, by_face, by_face[::-1].copy(), rng.permutation(n).astype(np.int32)):
        g = mg.point_mesh_backward(*args, order=None if order is None else dev(order, device))
        np.testing.assert_array_equal(host(g).astype(np.float64), want)


@pytest.mark.parametrize("na,nb", [(1, 1), (65, 300), (300, 0), (5000, 20000)])
def test_chamfer_backward_in_any_order(device, na, nb):
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(na + nb)
    a, b = (rng.integers(-4, 5, size=(3, n)).astype(np.float32) for n in (na, nb))
    ab = rng.integers(-1, nb, size=na).astype(np.int32) if nb else np.full(na, -1, np.int32)
    ba = rng.integers(-1, na, size=nb).astype(np.int32)
    want = np.zeros((3, na))
    i = np.flatnonzero(ab >= 0)
    want[:, i] += 2.0 * (a[:, i] - b[:, ab[i]])
    j = np.flatnonzero(ba >= 0)
    for c in range(3):
        np.add.at(want[c], ba[j], 4.0 * (a[c, ba[j]] - b[c, j]))
    args = tuple(dev(x, device) for x in (a, b, ab, ba))
    for order in (None, np.argsort(ba, kind="stable").astype(np.int32), rng.permutation(nb).astype(np.int32)):
        g = mg.chamfer_backward(*args, 1.0, 2.0, order_b=None if order is None else dev(order, device))
        np.testing.assert_array_equal(host(g).astype(np.float64), want)


def test_scatter_order_is_a_copy(device):
    import paper_2606_00444_amd as mg
    P = torch.rand(3, 20000, device=device)
    bvh = mg.lbvh_build(P, None)
    order = mg.scatter_order(bvh)
    kept = order.clone()
    mg.lbvh_build(P.flip(1).contiguous(), None, bvh=bvh)
    assert torch.equal(order, kept)
    assert mg.scatter_order(mg.lbvh_build(P[:, :100].contiguous(), None)) is None


@pytest.mark.parametrize("n", [1, 255, 8191, 8192, 8193, 300000])
def test_mean_forms(device, n):
    import paper_2606_00444_amd as mg
    x = np.random.default_rng(n).integers(-100, 100, size=n).astype(np.float32)
    assert host(mg.mean(dev(x, device)))[0] == x.astype(np.float64).sum() / n


@pytest.mark.parametrize("na,nb", [(1, 1), (70, 3000), (9000, 2047), (2049, 1100000)])
def test_chamfer_means(device, na, nb):
    import paper_2606_00444_amd as mg
    rng = np.random.default_rng(na)
    a, b = (dev(rng.integers(0, 40, size=(3, n)).astype(np.float32), device) for n in (na, nb))
    add = torch.tensor([0.5], dtype=torch.float64, device=device)
    o = mg.chamfer(a, mg.lbvh_build(a, None), b, mg.lbvh_build(b, None), add=add)
    ma, mb = (host(o[k]).astype(np.float64).sum() / n for k, n in (("d_ab", na), ("d_ba", nb)))
    assert host(o["loss"]).tolist() == [ma, mb, (ma + mb) + 0.5]
