"""One query per lane on either side of the tree size from which its bound takes the box's
ball in, and on a closed mesh of each, against all faces."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev
from synth.meshes import uv_sphere

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("n", [4100, 8191, 8192, 8193, 10200])
@pytest.mark.parametrize("offset", [0.0, 300.0])
def test_lane_matches_all_faces(device, n, offset):
    import paper_2606_00444_amd as mg
    v, f = uv_sphere(100, 52)
    V = np.ascontiguousarray((v + offset).T.astype(np.float32))
    F = np.ascontiguousarray(f.T.astype(np.int32))[:, :n]
    assert F.shape[1] == n
    rng = np.random.default_rng(n)
    Q = (np.concatenate([rng.uniform(-1.3, 1.3, size=(3, 700)), 0.01 * rng.normal(size=(3, 60))], axis=1) + offset).astype(np.float32)
    Vd, Fd, Qd = dev(V, device), dev(np.ascontiguousarray(F), device), dev(Q, device)
    ref = mg.closest_point_bruteforce(Vd, Fd, Qd, normal=True)
    bvh = mg.lbvh_build(Vd, Fd)
    for hint in (None, ref["face"].roll(1)):
        r = mg.closest_point_query(bvh, Vd, Qd, normal=True, kernel="lane", hint=hint)
        for key in ref:
            assert torch.equal(r[key], ref[key]), key
