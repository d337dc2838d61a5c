"""Runs whose random-walk steps add the moment partials themselves (32 partials
or fewer, of 128 particles each) give the proposal scales of the separate
moments kernels, to the bit: one partial, one past a partial, quarters of
unequal length, the last size that is added in the step and the first that is
not, by 16 and 32 wide moment matrices."""
import pytest
import torch

import paper_1304_4334_amd as S
import synthdata as SD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["egarch11", "egarch23"])
@pytest.mark.parametrize("J,N", [(2, 64), (3, 43), (4, 171), (4, 1024), (4, 1025)])
def test_step_adds_the_partials_of_a_small_population(name, J, N):
    w = SD.workload(name, T=120, J=J, N=N)
    m = S.Model.from_workload(w)
    pop = S.Population(m, J, N, max_chunk=32)
    rec = S.smc_run(m, pop, seed=5, Lmax=200, RmaxRec=64)
    # the first cycle again, call by call
    S.smc_init_from_prior(m, pop, 5)
    t, _, _ = S.smc_correct(m, pop, 0, w.T)
    assert t == rec.t_end[0]
    S.smc_resample(m, pop, seed=5, cycle=1)
    mh = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    for r in range(int(rec.R[0])):
        hl = S.smc_particle_moments(m, pop, mh)
        n = S.smc_mutate(m, pop, t, hl, 5, cycle=1, it=r + 1)
        S.smc_adapt_scale(n, pop.P, 250, mh)
        assert torch.equal(rec.hchol[0, r], hl), r
        assert int(n) == int(rec.n_accept[0, r]), r
