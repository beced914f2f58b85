"""The default queries per wave of the batch traversal, on the host, at the rule's edges."""

import ctypes

import pytest

from paper_2606_00444_amd import MG_PRIM_POINTS, MG_PRIM_TRIANGLES, _lib


def _default(kind, n):
    b = ctypes.c_int32(-1)
    return _lib.load().mg_query_default_batch(kind, n, ctypes.byref(b)), b.value


@pytest.mark.parametrize("n,tri,points", [(0, 1, 1), (1, 1, 1), (4095, 1, 1), (4096, 2, 2), (8191, 2, 2), (8192, 4, 4),
                                          (16383, 4, 4), (16384, 8, 8), (32767, 8, 8), (32768, 8, 16), (40960, 8, 16),
                                          (40961, 16, 16), (1000000, 16, 16)])
def test_rule(n, tri, points):
    assert _default(MG_PRIM_TRIANGLES, n) == (0, tri)
    assert _default(MG_PRIM_POINTS, n) == (0, points)


def test_bad_arguments():
    assert _default(7, 10)[0] == 1 and _default(MG_PRIM_POINTS, -1)[0] == 1
