"""The posterior report and the log marginal likelihood at the edges of their
kernels' tiles (64 groups a tile, groups held in registers up to 2,048
particles; rows of up to 2,047 groups in LDS, 4,096 values a tile), against
plain numpy in FP64.  Both sides are sums of at most 3e5 FP64 terms of one
scale, so they agree to about 3e5 eps = 7e-11 at worst: 1e-9 relative for the
moments (as the other report tests), 1e-11 for the log-ML, whose sums run over
at most 4,096 terms."""
import numpy as np
import pytest
import torch

import paper_1304_4334_amd as S
import synthdata as SD
from tests.gpu_helpers import gpu_model

pytestmark = pytest.mark.gpu


def report(x, J, N):
    g = x.reshape(-1, J, N)
    gj = g.mean(2)
    m = gj.mean(1)
    b = ((gj - m[:, None]) ** 2).sum(1)
    var = ((g - m[:, None, None]) ** 2).sum((1, 2)) / (J * N - 1)
    return np.stack([m, np.sqrt(var), np.sqrt(b / (J * (J - 1))), var / (N * b / (J - 1))], 1)


@pytest.mark.parametrize("J,N", [(2, 2), (63, 3), (64, 256), (65, 257), (130, 5), (3, 2047),
                                 (2, 2048), (66, 2049), (129, 1000)])
def test_parameter_report_at_tile_edges(J, N):
    gm = gpu_model(SD.workload("linreg"))
    pop = S.Population(gm, J, N, max_chunk=16)
    x = np.random.default_rng(J * 10007 + N).normal(1.0, 2.0, (gm.d, J * N))
    pop.theta.copy_(torch.from_numpy(x))
    want = report(x, J, N)
    got = S.smc_test_moments(gm, pop, 0, S.SMC_TEST_PARAMS).cpu().numpy()
    assert np.allclose(got, want, rtol=1e-9, atol=0.0)
    assert S.smc_rne(gm, pop).item() == pytest.approx(want[:, 3].mean(), rel=1e-9)


@pytest.mark.parametrize("L,J", [(1, 2), (50, 64), (63, 64), (64, 64), (257, 5), (300, 63),
                                 (3, 2047), (2, 2048), (4, 4096)])
def test_log_ml_at_tile_edges(L, J):
    g = np.random.default_rng(L * 5003 + J).normal(-40.0, 0.5 / np.sqrt(L), (L, J))
    s = g.sum(0)
    r = np.exp(s - s.max())
    want = [s.max() + np.log(r.mean()),
            np.sqrt(((r - r.mean()) ** 2).sum() / (J * (J - 1))) / r.mean(),
            (g.max(1) + np.log(np.exp(g - g.max(1)[:, None]).mean(1))).sum()]
    got = S.smc_log_ml(torch.from_numpy(g).cuda()).cpu().numpy()
    assert np.allclose(got, want, rtol=1e-11, atol=0.0)
