"""Adaptive batches that end with an error: a failed batch names the run that
failed and leaves nothing behind it (no work, no decision that would land among
those of a later batch), whichever stream the next one comes from."""
import numpy as np
import pytest
import torch

import paper_1304_4334_amd as S
import synthdata as SD

pytestmark = pytest.mark.gpu

SPECS = [("egarch11", 400, 4, 64, 0), ("egarch2t", 250, 4, 96, 1), ("egarch11", 700, 2, 200, 2),
         ("egarch2t", 333, 8, 32, 3), ("egarch11", 90, 2, 1000, 4), ("egarch11", 395, 2, 65, 6)]
SEEDS = [71, 72, 73, 74, 75, 76]


def _batch(specs, spoil=None):
    models, pops = [], []
    for i, (name, T, J, N, off) in enumerate(specs):
        w = SD.workload(name, T=T, J=J, N=N, seed_offset=off)
        y = np.array(w.y[:T], dtype=np.float64)
        if i == spoil:
            y[60] = np.nan  # every particle's weight is zero from date 61 on
        models.append(S.Model(w.kind, y, K=w.K, shock=w.shock, precision=S.SMC_FP32))
        pops.append(S.Population(models[-1], J, N, max_chunk=64))
    return models, pops


def _run(models, pops):
    recs = S.smc_run_batch(models, pops, SEEDS, Lmax=700, RmaxRec=64)
    return [r.summary()["log_ml"] for r in recs], [p.theta.clone() for p in pops]


@pytest.fixture(scope="module")
def want():
    models, pops = _batch(SPECS)
    out = _run(models, pops)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("spoil", [4, 2])
def test_failed_batch_leaves_nothing_behind(spoil, want):
    bad, good = _batch(SPECS, spoil), _batch(SPECS)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for rep in range(3):
        with torch.cuda.stream(streams[0]):
            with pytest.raises(S.SmcError) as ei:
                S.smc_run_batch(*bad, SEEDS, Lmax=700, RmaxRec=64)
            assert ei.value.status == S.SMC_E_NUMERIC
            assert f"run {spoil}:" in str(ei.value)
            # nothing is queued any more, neither there nor on any other lane
            assert streams[0].query()
        with torch.cuda.stream(streams[1]):  # other runs in other lanes
            ml, th = _run(*good)
        streams[1].synchronize()
        assert ml == want[0], rep
        assert all(torch.equal(a, b) for a, b in zip(th, want[1])), rep
