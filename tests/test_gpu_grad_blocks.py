"""Gradients by blocks of eight waves against one wave per 64 particles: the
same operations in the same order, so the same bits.  The same parameter
vectors are given alone (few particles: blocks) and repeated to 33,000
columns (one wave each); dates around the checkpoint segments (64 observations
in FP32, 32 in FP64) and the blocks' sub-blocks of 4 and 8."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1304_4334_amd as S
from paper_1304_4334_amd import autograd as A
import synthdata as SD
from tests.gpu_helpers import gpu_model, ora_model

pytestmark = pytest.mark.gpu

MANY = 33000


def workload(name, T):
    if name in ("egarch1t", "egarch2g"):
        K = 1 if name == "egarch1t" else 2
        th = SD.egarch2t_truth()
        th = th[[0, 1, 2, 4, 6, 8]] if K == 1 else th[:8]
        sh = SD.STUDENT_T if K == 1 else SD.GAUSS
        return SD.Workload(name, SD.EGARCH, K=K, shock=sh, T=T, J=2, N=64, theta_true=th,
                           y=SD.egarch_series(th, T, K, sh, 11))
    return SD.workload(name, T=T)


@pytest.mark.parametrize("prec", [S.SMC_FP64, S.SMC_FP32])
@pytest.mark.parametrize("name", ["egarch11", "egarch2g", "egarch1t", "egarch2t", "egarch12",
                                  "egarch23", "egarch34"])
def test_blocks_equal_single_waves(name, prec):
    w = workload(name, 203)
    m = gpu_model(w, prec)
    P = 65
    th = torch.from_numpy(SD.random_thetas(w, P, 5, spread=0.1).T.copy()).cuda()
    wt = torch.from_numpy(np.random.default_rng(1).uniform(-1.0, 2.0, P)).cuda()
    many = th.repeat(1, MANY // P + 1)
    wmany = wt.repeat(MANY // P + 1)
    for t in (1, 3, 4, 5, 8, 9, 31, 32, 33, 36, 63, 64, 65, 72, 127, 128, 129, 192, 203):
        g = S.smc_loglik_backward(m, th, t, wt)
        g1 = S.smc_loglik_backward(m, many, t, wmany)
        assert torch.isfinite(g).all()
        assert torch.equal(g, g1[:, :P]), (t, (g - g1[:, :P]).abs().max().item())
        assert torch.equal(g1[:, :P], g1[:, -P:])
        # the pair that keeps the checkpoints: smc_loglik's values, and the
        # gradients (FP64 Student-t: another order of the density terms' sum, so
        # 1e-13 of the largest entry, far above the 1e-16 of a reordered sum)
        ll, ck = S.smc_loglik_ckpt(m, th, t)
        ll1, ck1 = S.smc_loglik_ckpt(m, many, t)
        assert torch.equal(ll, S.smc_loglik(m, th, t)) and torch.equal(ll, ll1[:P])
        h = S.smc_loglik_backward_ckpt(m, th, t, wt, ck)
        h1 = S.smc_loglik_backward_ckpt(m, many, t, wmany, ck1)
        assert torch.equal(h, h1[:, :P])
        assert (h - g).abs().max() <= 1e-13 * g.abs().max()
        assert torch.equal(h, S.smc_loglik_backward_ckpt(m, th, t, wt, ck))


def test_autograd_runs_forward_once_and_back_twice():
    """The autograd function: values of smc_loglik with and without a gradient
    wanted, the gradient of smc_loglik_backward (1e-13, see above), a graph kept
    for a second backward, saved-tensor hooks passed by, the regression."""
    for name in ("egarch2t", "linreg"):
        m = gpu_model(SD.workload(name, T=120))
        x = torch.from_numpy(SD.random_thetas(SD.workload(name, T=120), 70, 2, spread=0.05).T.copy())
        x = x.cuda()
        w = torch.linspace(0.5, 1.5, 70, dtype=torch.float64, device="cuda")
        want = S.smc_loglik_backward(m, x, 120, w)
        assert torch.equal(A.loglik(x, m, 120), S.smc_loglik(m, x, 120))
        th = x.clone().requires_grad_(True)
        seen = []
        with torch.autograd.graph.saved_tensors_hooks(lambda v: (seen.append(1), v.cpu())[1],
                                                      lambda v: v.cuda()):
            ll = A.loglik(th, m, 120)
        assert len(seen) == 2 and torch.equal(ll, S.smc_loglik(m, x, 120))
        for _ in range(2):
            (g,) = torch.autograd.grad(ll, th, w, retain_graph=True)
            assert (g - want).abs().max() <= 1e-13 * want.abs().max()


@pytest.mark.parametrize("prec", [S.SMC_FP64, S.SMC_FP32])
@pytest.mark.parametrize("name", ["egarch11", "egarch2t", "egarch23"])
def test_langevin_blocks_equal_single_waves(name, prec):
    """The Langevin step's proposals depend on the particle's index, so the
    first 2 x 70 of a population of 2 x 70 and of 472 x 70 are compared (groups
    do not enter the step)."""
    w = workload(name, 100)
    m = gpu_model(w, prec)
    th = torch.from_numpy(SD.random_thetas(w, 140, 5, spread=0.05).T.copy()).cuda()
    lp = torch.from_numpy(np.array([O.logprior(ora_model(w), x) for x in th.cpu().numpy().T])).cuda()
    eye = torch.eye(m.d, dtype=torch.float64, device="cuda")
    out = []
    for J in (2, 472):
        pop = S.Population(m, J, 70, max_chunk=16, with_grad=True)
        pop.theta.copy_(th.repeat(1, J // 2))
        pop.loglik.copy_(S.smc_loglik(m, pop.theta, 77, state_out=pop.state))
        pop.logprior.copy_(lp.repeat(J // 2))
        S.smc_posterior_grad(m, pop, 77)
        acc = torch.zeros((3, pop.P), dtype=torch.uint8, device="cuda")
        n = torch.zeros(1, dtype=torch.int64, device="cuda")
        for it, h in enumerate((0.01, 0.1, 0.5)):  # nearly all accepted to nearly none
            S.smc_mutate(m, pop, 77, h * eye, 9, cycle=1, it=it + 1, kernel=S.SMC_KERNEL_MALA,
                         n_accept=n, accepted=acc[it])
        assert 0 < acc.sum().item() < acc.numel() and n.item() == acc.sum().item()
        out.append([x[..., :140].clone() for x in (pop.theta, pop.logprior, pop.loglik, pop.state,
                                                   pop.grad, acc)])
    for a, b in zip(*out):
        assert torch.equal(a, b)
