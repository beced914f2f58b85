"""The batched launch's queries per wave, on the host: a number that a scene or the plan
names is taken as it is, and the default follows the queries that a tile holds."""

import ctypes

import pytest

from paper_2606_00444_amd import _lib


def _per_wave(n_queries, batch=0, tile=0, plan_batch=0, plan_tile=0, options=True):
    s, o, out = _lib.BatchScene(), _lib.BatchOptions(), ctypes.c_int32(-1)
    s.n_queries, s.batch, s.query_tile = n_queries, batch, tile
    o.batch, o.query_tile = plan_batch, plan_tile
    st = _lib.load().mg_batch_queries_per_wave(ctypes.byref(s), ctypes.byref(o) if options else None, ctypes.byref(out))
    return st, out.value


@pytest.mark.parametrize("batch", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("tile", [64, 256, 1024])
def test_a_named_number_is_taken(batch, tile):
    assert _per_wave(60000, batch=batch, tile=tile) == (0, batch)
    assert _per_wave(60000, plan_batch=batch, plan_tile=tile) == (0, batch)
    assert _per_wave(60000, batch=batch, plan_batch=16, plan_tile=tile) == (0, batch)      # the scene's before the plan's


@pytest.mark.parametrize("n,tile,want", [(60000, 0, 16), (60000, 16, 4), (60000, 32, 8), (60000, 48, 16), (60000, 64, 16),
                                         (64, 256, 16), (33, 256, 16), (32, 256, 8), (17, 256, 8), (16, 256, 4),
                                         (1, 256, 4), (0, 256, 4)])
def test_the_default_runs_a_tile_at_once(n, tile, want):
    assert _per_wave(n, tile=tile) == (0, want)
    assert _per_wave(n, plan_tile=tile) == (0, want)
    if tile == 0:
        assert _per_wave(n, options=False) == (0, want)


def test_what_is_refused():
    for kw in ({"batch": 3}, {"batch": 32}, {"plan_batch": -1}, {"batch": 16, "tile": 32}, {"tile": 24}, {"tile": -64}):
        assert _per_wave(1000, **kw)[0] == 1, kw
