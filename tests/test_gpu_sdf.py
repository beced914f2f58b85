"""Index signed-distance grid on the GPU against the float64 oracle."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev, host, scale_of
from synth import make_config
from oracle import sdf as osdf
from oracle import knn as ok

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


def _grid_for(V, res, grow=0.2):
    lo, hi = V.min(1), V.max(1)
    pad = grow * (hi - lo)
    lo, hi = lo - pad, hi + pad
    h = float((hi - lo).max() / (res - 1))
    dims = tuple(int(np.ceil((hi[a] - lo[a]) / h)) + 1 for a in range(3))
    return tuple(float(x) for x in lo), h, dims


def _check_grid(V, F, sdf_dev, face_dev, face_k, lo, h, dims):
    """The device field against the oracle evaluated with the device's stored faces."""
    L = scale_of(V)
    P = osdf.grid_points(lo, h, dims)
    ref = osdf.sdf_from_faces(V, F, P, face_k)
    got = sdf_dev.astype(np.float64)
    tol = 1e-5 * np.maximum(np.abs(ref["sdf"]), 0.1 * L)
    # magnitudes always agree; a sign may flip only where the distance is ~0
    assert (np.abs(np.abs(got) - np.abs(ref["sdf"])) <= tol).all()
    flip = np.sign(got) != np.sign(ref["sdf"])
    assert (np.abs(ref["sdf"][flip]) <= tol[flip]).all()
    # the winning face: the oracle's, or a tie at the same distance (a node whose nearest
    # feature is a vertex or an edge is equally near every face around it)
    diff = face_dev != ref["face"]
    if diff.any():
        from oracle import closest as oc
        d = np.sqrt(oc.closest_on_faces(V, F, P[:, diff], face_dev[diff])["dist2"])
        assert (np.abs(d - np.abs(ref["sdf"][diff])) <= tol[diff]).all()
    return ref


def test_sdf_small_template_and_frames(device):
    import paper_2606_00444_amd as mg
    from paper_2606_00444_amd.sdf import IndexSDF
    sc = make_config(2, small=True)
    V0, F = sc.verts0, sc.faces
    lo, h, dims = _grid_for(V0, 24)
    S = IndexSDF(dev(V0, device), dev(F, device), lo, h, dims, k=4)
    # node positions
    np.testing.assert_allclose(host(S.points), osdf.grid_points(lo, h, dims), rtol=0, atol=1e-6 * scale_of(V0))
    # stored faces: the k nearest template faces (distances unique, faces up to ties)
    P = osdf.grid_points(lo, h, dims)
    ref_f, ref_d2 = ok.knn_faces(V0, F, P, 4)
    fk = host(S.face_k).astype(np.int64)
    from oracle import closest as oc
    for j in range(4):
        d = np.sqrt(oc.closest_on_faces(V0, F, P, fk[j])["dist2"])
        assert (np.abs(d - np.sqrt(ref_d2[j])) <= 1e-5 * np.maximum(np.sqrt(ref_d2[j]), 0.1 * scale_of(V0))).all()
    # frame 0 pose (the template): the exact signed distance field
    S.update(dev(V0, device))
    ref = _check_grid(V0, F, host(S.sdf), host(S.face), fk, lo, h, dims)
    allf = np.repeat(np.arange(F.shape[1])[:, None], P.shape[1], axis=1)
    exact = osdf.sdf_from_faces(V0, F, P, allf)
    L = scale_of(V0)
    assert (np.abs(np.abs(ref["sdf"]) - np.abs(exact["sdf"])) <= 1e-5 * np.maximum(np.abs(exact["sdf"]), 0.1 * L)).all()
    # later frames with the same stored faces
    for t in (20, 110):
        Vt = sc.frames([t])[0]
        S.update(dev(Vt, device))
        _check_grid(Vt, F, host(S.sdf), host(S.face), fk, lo, h, dims)
        # trilinear sampling of the device grid
        rng = np.random.default_rng(t)
        Q = (np.array(lo)[:, None] + rng.random((3, 3000)) * (h * (np.array(dims) - 1))[:, None]).astype(np.float32)
        Q = np.concatenate([Q, np.array([[lo[0] - h], [lo[1]], [lo[2]]], np.float32)], axis=1)   # one outside
        got = host(S.sample(dev(Q, device)))
        want = osdf.sample(host(S.sdf), lo, h, dims, Q)
        assert np.isinf(got[-1]) and np.isinf(want[-1])
        np.testing.assert_allclose(got[:-1], want[:-1], rtol=1e-5, atol=1e-6 * scale_of(Vt))


def test_sdf_full_size_template(device):
    """The 40,000-face template on a 40^3 grid, frame 150, k = 4."""
    from paper_2606_00444_amd.sdf import IndexSDF
    sc = make_config(2)
    lo, h, dims = _grid_for(sc.verts0, 40)
    S = IndexSDF(dev(sc.verts0, device), dev(sc.faces, device), lo, h, dims, k=4)
    Vt = sc.frames([150])[0]
    S.update(dev(Vt, device))
    _check_grid(Vt, sc.faces, host(S.sdf), host(S.face), host(S.face_k).astype(np.int64), lo, h, dims)


def test_sdf_ignores_invalid_face_ids(device):
    import paper_2606_00444_amd as mg
    from paper_2606_00444_amd.sdf import IndexSDF
    sc = make_config(1, small=True)
    lo, h, dims = _grid_for(sc.verts0, 8)
    S = IndexSDF(dev(sc.verts0, device), dev(sc.faces, device), lo, h, dims, k=2)
    S.face_k[1].fill_(10 ** 6)                       # slot 1 out of range everywhere
    S.face_k[0, :5].fill_(-1)                        # five nodes with no valid face
    S.update(dev(sc.verts0, device))
    sdf = host(S.sdf)
    assert np.isinf(sdf[:5]).all() and np.isfinite(sdf[5:]).all()
    assert (host(S.face)[:5] == -1).all()


@pytest.mark.parametrize("k", [1, 2, 4, 8])
@pytest.mark.parametrize("short", [0, 1])
def test_sdf_face_records_change_nothing(device, k, short):
    """mg_sdf_update_records at the node count from which it writes the faces' corners
    (2^19 stored ids, not a whole number of workgroups) and just below, with records that
    are long enough or one float short: mg_sdf_update's values, and ids outside the mesh
    ignored."""
    import ctypes
    from paper_2606_00444_amd import _lib
    from paper_2606_00444_amd.api import _ptr, _stream
    rng = np.random.default_rng(k)
    nv, nf = 301, 599
    V = dev(rng.normal(size=(3, nv)).astype(np.float32), device)
    F = dev(rng.integers(0, nv, size=(3, nf)).astype(np.int32), device)
    lib = _lib.load()
    rec = torch.empty(12 * nf - short, device=device)
    for nz in (2 ** 19 // k // 1024, 2 ** 19 // k // 1024 + 1):
        dims = (31, 33, nz)                        # 1023 a layer: just below, and just above
        n = dims[0] * dims[1] * dims[2]
        face_k = torch.randint(-1, nf + 1, (k, n), dtype=torch.int32, device=device)
        out = []
        for records, size in ((None, 0), (_ptr(rec), 4 * rec.numel())):
            d, w = torch.empty(n, device=device), torch.empty(n, dtype=torch.int32, device=device)
            st = lib.mg_sdf_update_records(_ptr(V), nv, _ptr(F), nf, _ptr(face_k), k, -1.0, -1.0, -1.0, 0.05, *dims,
                                           _ptr(d), _ptr(w), records, ctypes.c_size_t(size), _stream())
            assert st == 0
            out.append((d, w))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
