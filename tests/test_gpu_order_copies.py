"""The autograd losses copy a processing order only for a gradient that will be asked for."""

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def device():
    return need_gpu()


@pytest.mark.parametrize("grad_a,grad_b", [(True, True), (True, False), (False, True), (False, False)])
def test_chamfer_copies_the_orders_its_gradients_use(device, monkeypatch, grad_a, grad_b):
    """One copy of the other set's Morton order for each input that needs a gradient, and the
    same gradients as with both."""
    from paper_2606_00444_amd import api, autograd
    calls = []
    monkeypatch.setattr(api, "scatter_order", lambda bvh, f=api.scatter_order: calls.append(bvh.n) or f(bvh))
    rng = np.random.default_rng(3)
    na, nb = 20000, 17000
    A, B = (dev(rng.integers(0, 40, size=(3, n)).astype(np.float32), device) for n in (na, nb))
    a, b = A.clone().requires_grad_(), B.clone().requires_grad_()
    autograd.ChamferLoss.apply(a, b).backward()
    both = (a.grad, b.grad)
    calls.clear()
    a, b = A.clone().requires_grad_(grad_a), B.clone().requires_grad_(grad_b)
    loss = autograd.ChamferLoss.apply(a, b)
    assert sorted(calls) == sorted([nb] * grad_a + [na] * grad_b)
    if grad_a or grad_b:
        loss.backward()
    # sums of some 50 terms under 1e-3 in another order: 50 additions' rounding of at most 0.05
    for x, needs, want in ((a, grad_a, both[0]), (b, grad_b, both[1])):
        assert x.grad is None if not needs else torch.allclose(x.grad, want, rtol=0, atol=2e-7)


def test_projection_loss_copies_no_order_without_a_gradient(device, monkeypatch):
    from paper_2606_00444_amd import api, autograd
    import paper_2606_00444_amd as mg
    from synth import make_config
    calls = []
    monkeypatch.setattr(api, "scatter_order", lambda bvh, f=api.scatter_order: calls.append(bvh.n) or f(bvh))
    sc = make_config(1, small=True)
    V, F = dev(sc.verts0, device), dev(sc.faces, device)
    binding = {k: dev(x, device) for k, x in sc.binding.items()}
    Y = dev(np.random.default_rng(4).normal(size=(3, 20000)).astype(np.float32), device)
    bvh = mg.lbvh_build(V, F)
    for needs in (False, True):
        calls.clear()
        autograd.template_projection_loss(V.clone().requires_grad_(needs), F, binding, Y, bvh)
        assert calls == [20000] * needs
