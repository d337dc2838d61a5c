"""The autograd likelihood where the device has no memory for checkpoints that
live as long as the graph: the value and the gradient are there all the same,
and the graph holds theta alone."""
import pytest
import torch

from paper_1304_4334_amd import _lib, autograd


def _no_room(*args, **kwargs):
    raise torch.OutOfMemoryError("no room for the checkpoints")


def test_forward_without_room_for_checkpoints(monkeypatch):
    """The calls replaced by plain functions of theta (CPU)."""
    monkeypatch.setattr(_lib, "smc_loglik_ckpt", _no_room)
    monkeypatch.setattr(_lib, "smc_loglik", lambda m, th, t: (t * th ** 2).sum(0))
    monkeypatch.setattr(_lib, "smc_loglik_backward", lambda m, th, t, dl: 2 * t * th * dl)
    th = torch.arange(6.0, dtype=torch.float64).reshape(2, 3).requires_grad_(True)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda v: (seen.append(v.shape), v)[1],
                                                  lambda v: v):
        ll = autograd.loglik(th, None, 5)
    assert seen == [th.shape]
    assert torch.equal(ll, (5 * th ** 2).sum(0))
    w = torch.tensor([1.0, -2.0, 0.5], dtype=torch.float64)
    for _ in range(2):
        (g,) = torch.autograd.grad(ll, th, w, retain_graph=True)
        assert torch.equal(g, 10 * th * w)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["egarch11", "egarch2t", "egarch23", "linreg"])
def test_gradient_without_room_for_checkpoints(name, monkeypatch):
    """The gradient of the two forms differs by 1e-13 of its size (their
    forward sweeps add in different groups)."""
    import synthdata as SD
    from tests.gpu_helpers import gpu_model

    w = SD.workload(name, T=120)
    m = gpu_model(w)
    th = torch.from_numpy(SD.random_thetas(w, 70, 2, spread=0.05).T.copy()).cuda()
    th.requires_grad_(True)
    wt = torch.linspace(0.5, 1.5, 70, dtype=torch.float64, device="cuda")
    ll = autograd.loglik(th, m, 120)
    (g,) = torch.autograd.grad(ll, th, wt)
    monkeypatch.setattr(_lib, "smc_loglik_ckpt", _no_room)
    ll1 = autograd.loglik(th, m, 120)
    (g1,) = torch.autograd.grad(ll1, th, wt)
    assert torch.equal(ll, ll1)
    assert (g - g1).abs().max() <= 1e-13 * g.abs().max()
