"""Refits of trees with 2048-leaf subtrees to other vertices than the build's, bitwise
against the oracle's refit of the same topology: 1024-thread workgroups with the top nodes
in LDS (one and two a thread) and, beyond 2,048 of them, in global scratch."""

import ctypes

import numpy as np
import pytest

from gpu_helpers import need_gpu, dev, decode_bvh
from oracle import lbvh as ol
from paper_2606_00444_amd._lib import LbvhHeader

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


def _points_of(codes):
    """The centre of each Morton cell of the unit cube."""
    out = np.zeros((3, codes.size))
    for axis in range(3):
        for i in range(10):
            out[axis] += ((codes >> (3 * i + 2 - axis)) & 1) << i
    return (out + 0.5) / 1024


def _combs():
    """256 cells of 2,060 points each, with a lone point in the sibling cell of each of the 22
    levels above the cell: every one of those levels is a top node with one leaf to a side."""
    cell = np.arange(256) << 22
    lone = (cell[:, None] | (1 << np.arange(22))).ravel()
    codes = np.concatenate([np.repeat(cell, 2060), lone])
    P = _points_of(np.random.default_rng(5).permutation(codes))
    return np.concatenate([P, [[0, 1], [0, 1], [0, 1]]], axis=1).astype(np.float32)


def _case(name):
    rng = np.random.default_rng(len(name))
    if name == "combs":
        return _combs(), None, (2049, 1 << 30)
    n = 524289 if name == "faces" else 1400000
    P = (rng.normal(size=(3, n + 2 if name == "faces" else n)) ** 3).astype(np.float32)
    F = np.stack([np.arange(n), np.arange(n) + 1, np.arange(n) + 2]).astype(np.int32) if name == "faces" else None
    return P, F, (1, 1024) if name == "faces" else (1025, 2048)


@pytest.mark.parametrize("name", ["faces", "points", "combs"])
def test_refit_to_other_vertices(device, name):
    import paper_2606_00444_amd as mg
    P, F, (least, most) = _case(name)
    print(f"refit: {name}, {P.shape[1]} vertices", flush=True)
    bvh = mg.lbvh_build(dev(P, device), None if F is None else dev(F, device))
    hdr = LbvhHeader.from_buffer_copy(bvh.buf[:ctypes.sizeof(LbvhHeader)].cpu().numpy().tobytes())
    assert hdr.chunk_log2 == 11 and least <= hdr.n_top <= most
    built = decode_bvh(bvh)
    ref = ol.build(P, F)
    np.testing.assert_array_equal(built["child"], ref["tree"]["child"])
    np.testing.assert_array_equal(built["internal_box"], ref["internal_box"])
    moved = (P[::-1] + np.random.default_rng(1).normal(size=P.shape)).astype(np.float32)
    for V in (moved, P):                              # away, and back again
        mg.lbvh_refit(bvh, dev(V, device))
        got = decode_bvh(bvh)
        leaf = ol.leaf_boxes(V, F, ref["perm"])
        box = ol.refit(ref["tree"], leaf)
        assert got["status"] == 0
        np.testing.assert_array_equal(got["leaf_box"], leaf)
        np.testing.assert_array_equal(got["internal_box"], box)
        np.testing.assert_array_equal(got["root_box"], box[0])
        np.testing.assert_array_equal(got["child"], ref["tree"]["child"])
