"""Launch shapes of the random-walk step for the families whose densities go to
waves of their own up to kSplitMaxP particles (launch.h), where the shape has no
effect: populations just above that limit step and run to the default shape's
bits in every shape, with the proposal scale passed in and folded into the
step."""
import os
import re

import numpy as np
import pytest
import torch

import oracle as O
import paper_1304_4334_amd as S
import synthdata as SD
from tests.gpu_helpers import theta_np

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(b, u) for b in (64, 128, 256) for u in (4, 8, 16)]
PAIRS = [("egarch2t", S.SMC_FP64), ("egarch23", S.SMC_FP32), ("egarch23", S.SMC_FP64)]
J, N = 33, 999  # ragged blocks for every shape


def _above_the_limit():
    src = open(os.path.join(ROOT, "paper_1304_4334_amd", "csrc", "launch.h")).read()
    limit = int(re.search(r"kSplitMaxP = (\d+);", src).group(1))
    assert J * N > limit, "the populations here must be stepped in the shape that is set"


@pytest.mark.parametrize("name,prec", PAIRS)
def test_every_shape_steps_to_the_same_bits(name, prec):
    _above_the_limit()
    w = SD.workload(name, T=517)
    m = S.Model(w.kind, w.y[:w.T], K=w.K, shock=w.shock, precision=prec, I=w.I)
    th = SD.random_thetas(w, N, 5, spread=0.02)
    om = O.Model.from_workload(w)
    lp = torch.tensor([O.logprior(om, x) for x in th], dtype=torch.float64).cuda().repeat(J)
    theta = torch.from_numpy(th.T.copy()).cuda().repeat(1, J)
    hl = torch.from_numpy(np.linalg.cholesky(np.cov(th.T)) * 0.1).cuda()
    # 64 and 63 whole groups of 8 observations, then 3 and 7 of a group
    for t in (517, 509, 511):
        ll = S.smc_loglik(m, theta, t)
        ref = None
        for b, u in [(64, 8)] + [x for x in SHAPES if x != (64, 8)]:
            m.set_launch(b, u)
            g = S.Population(m, J, N, max_chunk=16)
            g.theta.copy_(theta)
            g.loglik.copy_(ll)
            g.logprior.copy_(lp)
            g.state.zero_()
            acc = torch.zeros(J * N, dtype=torch.uint8, device="cuda")
            n = S.smc_mutate(m, g, t, hl, seed=3, cycle=2, it=1, accepted=acc)
            out = (g.theta, g.logprior, g.loglik, g.state, acc, n)
            if ref is None:
                ref = out
                assert 0 < n.item() < J * N and n.item() == acc.sum().item()
            for a, r in zip(out, ref):
                assert torch.equal(a, r), (t, b, u)


@pytest.mark.parametrize("name,prec", PAIRS)
def test_adaptive_run_in_any_shape_is_the_same_run(name, prec):
    _above_the_limit()
    w = SD.workload(name, T=100)
    m = S.Model(w.kind, w.y[:w.T], K=w.K, shock=w.shock, precision=prec, I=w.I)
    res = {}
    for b, u in ((64, 8), (128, 4), (256, 16)):
        m.set_launch(b, u)
        g = S.Population(m, J, N, max_chunk=32)
        s = S.smc_run(m, g, seed=9, Lmax=100, RmaxRec=64).summary()
        res[(b, u)] = (s, theta_np(g))
    a, tha = res[(64, 8)]
    assert a["L"] > 1 and 0 < a["n_accept"].sum()
    for k, (s, th) in res.items():
        assert np.array_equal(s["t_end"], a["t_end"]) and np.array_equal(s["R"], a["R"]), k
        assert np.array_equal(s["n_accept"], a["n_accept"]), k
        assert s["log_ml"] == a["log_ml"] and s["nse"] == a["nse"], k
        assert np.array_equal(th, tha), k
