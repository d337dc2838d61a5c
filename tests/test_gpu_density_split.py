"""Likelihoods and random-walk steps whose densities are evaluated by waves of
their own (few particles) against those of one wave per 64 particles (the same
particles repeated to more than 32,768): the same operations in the same
order, so the same bits.  Dates around the spans of 8 (FP64) and 16 (FP32)
observations and the stages of three spans."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1304_4334_amd as S
import synthdata as SD
from tests.gpu_helpers import gpu_model, ora_model

pytestmark = pytest.mark.gpu

CASES = [("egarch2t", S.SMC_FP64), ("egarch12", S.SMC_FP64), ("egarch23", S.SMC_FP64),
         ("egarch44", S.SMC_FP64), ("egarch12", S.SMC_FP32), ("egarch23", S.SMC_FP32),
         ("egarch44", S.SMC_FP32)]


@pytest.mark.parametrize("name,prec", CASES)
def test_likelihood_equals_single_waves(name, prec):
    w = SD.workload(name, T=151)
    m = gpu_model(w, prec)
    P = 130
    th = torch.from_numpy(SD.random_thetas(w, P, 3, spread=0.1).T.copy()).cuda()
    many = th.repeat(1, 33000 // P + 1)
    for t in (1, 2, 8, 9, 16, 17, 23, 24, 25, 26, 32, 33, 47, 48, 49, 50, 57, 64, 65, 72, 73, 96, 97,
              98, 144, 145, 151):
        st, st1 = (torch.zeros((m.S, x.shape[1]), dtype=m.state_dtype, device="cuda")
                   for x in (th, many))
        ll = S.smc_loglik(m, th, t, state_out=st)
        ll1 = S.smc_loglik(m, many, t, state_out=st1)
        assert torch.isfinite(ll).all()
        assert torch.equal(ll, ll1[:P]) and torch.equal(st, st1[:, :P]), t


@pytest.mark.parametrize("name,prec", CASES)
def test_step_equals_single_waves(name, prec):
    """Proposals depend on the particle's index: the first 2 x 70 of 2 x 70 and
    of 472 x 70 particles, at dates below and above a stage."""
    w = SD.workload(name, T=100)
    m = gpu_model(w, prec)
    th = torch.from_numpy(SD.random_thetas(w, 140, 5, spread=0.05).T.copy()).cuda()
    lp = torch.from_numpy(np.array([O.logprior(ora_model(w), x) for x in th.cpu().numpy().T])).cuda()
    eye = torch.eye(m.d, dtype=torch.float64, device="cuda")
    for t in (5, 100):
        out = []
        for J in (2, 472):
            pop = S.Population(m, J, 70, max_chunk=16)
            pop.theta.copy_(th.repeat(1, J // 2))
            pop.logprior.copy_(lp.repeat(J // 2))
            pop.loglik.copy_(S.smc_loglik(m, pop.theta, t, state_out=pop.state))
            acc = torch.zeros((3, pop.P), dtype=torch.uint8, device="cuda")
            n = torch.zeros(1, dtype=torch.int64, device="cuda")
            for it, h in enumerate((0.01, 0.1, 1.0)):  # nearly all accepted to nearly none
                S.smc_mutate(m, pop, t, h * eye, 9, cycle=1, it=it + 1, n_accept=n, accepted=acc[it])
            assert 0 < acc.sum().item() < acc.numel() and n.item() == acc.sum().item()
            out.append([x[..., :140].clone() for x in (pop.theta, pop.logprior, pop.loglik,
                                                       pop.state, acc)])
        for a, b in zip(*out):
            assert torch.equal(a, b)
