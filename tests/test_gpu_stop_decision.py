"""The stopping decision made in the commit's launch: chunks of up to 1,024
checked dates (two rounds of 512 RSS values a wave, eight loads of a lane in
flight) stop where chunks of at most 16 do, whose values one load covers, and
where the device-driven chunks' own decision kernel stops."""
import pytest
import torch

import paper_1304_4334_amd as S
import synthdata as SD

pytestmark = pytest.mark.gpu

T = 2100


@pytest.fixture(scope="module")
def model():
    return S.Model.from_workload(SD.workload("egarch11", T=T, J=2, N=100))


def _pop(m, max_chunk):
    pop = S.Population(m, 2, 100, max_chunk=max_chunk)
    S.smc_init_from_prior(m, pop, 3)
    # particles close to their mean: the RSS falls over hundreds of dates
    mean = pop.theta.mean(dim=1, keepdim=True)
    pop.theta.copy_(mean + 0.02 * (pop.theta - mean))
    return pop


@pytest.mark.parametrize("check_every", [1, 3])
@pytest.mark.parametrize("rss_min", [1.5, 0.995, 0.97, 0.9, 0.7, 0.4, 0.2, 1e-6])
def test_long_chunks_stop_where_short_ones_do(model, check_every, rss_min):
    want_t, want_rss, _ = S.smc_correct(model, _pop(model, 16), 0, T, check_every, rss_min)
    for max_chunk in (65, 511, 1024):
        t, rss, _ = S.smc_correct(model, _pop(model, max_chunk), 0, T, check_every, rss_min)
        assert t == want_t
        # sums of up to 2,100 rounded terms, in chunks of another length
        assert rss == pytest.approx(want_rss, rel=1e-9)
    t_dev, rss_dev = S.smc_correct_async(model, _pop(model, 1024), 0, T, check_every, rss_min)[:2]
    torch.cuda.synchronize()
    assert int(t_dev) == want_t and float(rss_dev) == pytest.approx(want_rss, rel=1e-9)
