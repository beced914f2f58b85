"""Cold nearest-point queries: what they search of the tree, walk included."""

import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("batch", [1, 4, 16, 32])
@pytest.mark.parametrize("n,most", [(5000, 40), (100000, 52)])
def test_a_cold_query_walks_one_path(device, n, most, batch):
    """Uniform points and queries: a walk by one node a level and the search after it expand
    some 35 and 45 nodes a query; a second node on every level makes that 45 and 60."""
    import paper_2606_00444_amd as mg
    g = torch.Generator(device=device).manual_seed(1)
    P = torch.rand(3, n, device=device, generator=g)
    Q = torch.rand(3, 4000, device=device, generator=g)
    bvh = mg.lbvh_build(P)
    c = torch.zeros(4, dtype=torch.int64, device=device)
    i, d = mg.nearest_point_query(bvh, P, Q, kernel="batch", batch=batch, seed=True, counters=c)
    assert c[0].item() <= most * 4000 and c[3].item() == 4000
    j, e = mg.nearest_point_query(bvh, P, Q, kernel="lane")
    assert torch.equal(i, j) and torch.equal(d, e)
