"""Every batch size of the batched launch in the tiles where it runs: tiles of one round
of the four waves and of a few, a ragged last tile, scenes shorter than a tile, and the
default's choice beside them."""

import pytest
import torch

from gpu_helpers import need_gpu
from test_gpu_batch import _compare, _scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("batch,tile", [(1, 4), (1, 12), (2, 8), (4, 16), (8, 32), (1, 256), (2, 256), (4, 256),
                                        (8, 256), (16, 64), (0, 16), (0, 48), (0, 256)])
def test_named_batches_in_small_tiles(device, batch, tile):
    import paper_2606_00444_amd as mg
    from paper_2606_00444_amd.batch import BatchPlan
    scenes = _scenes(device, frames=2)
    for (s, _, _), n in zip(scenes, (1, 31, 333)):
        s["queries"] = s["queries"][:, :n].contiguous()
    for seed in (False, True):
        print(f"batched: batch {batch}, tile {tile}, seed {seed}", flush=True)
        plan = BatchPlan([s for s, _, _ in scenes], batch=batch, seed=seed, query_tile=tile)
        plan.run()
        torch.cuda.synchronize()
        assert plan.status() == 0
        _compare(mg, scenes, plan, {"batch": 4, "seed": seed})
