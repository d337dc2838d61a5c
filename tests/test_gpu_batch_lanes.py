"""Adaptive batches with several runs to a lane (more runs than lanes, uneven
lanes, runs of different lengths and sizes), so that one persistent launch
holds items of several runs, some lanes hold several pending decisions, and a
run's C phase stands beside another's M phase: each run equals the same run on
its own."""
import numpy as np
import pytest
import torch

import paper_1304_4334_amd as S
import synthdata as SD
from tests.gpu_helpers import theta_np

pytestmark = pytest.mark.gpu

# lanes hold runs of similar cost per iteration (T x K): 3, 2, 3 and 2 of them
SPECS = [("egarch11", 400, 4, 64, 0), ("egarch2t", 250, 4, 96, 1), ("egarch11", 700, 2, 200, 2),
         ("egarch2t", 333, 8, 32, 3), ("egarch11", 90, 2, 1000, 4), ("egarch2t", 120, 3, 333, 5),
         ("egarch11", 395, 2, 65, 6), ("egarch2t", 340, 4, 300, 7), ("egarch11", 120, 5, 77, 8),
         ("egarch11", 41, 4, 128, 9)]
SEEDS = list(range(51, 51 + len(SPECS)))


def _runs(prec, specs=SPECS, with_grad=False, shape=None):
    out = []
    for name, T, J, N, off in specs:
        w = SD.workload(name, T=T, J=J, N=N, seed_offset=off)
        m = S.Model(w.kind, w.y[:T], K=w.K, shock=w.shock, precision=prec)
        if shape:
            m.set_launch(*shape)
        out.append((w, m, S.Population(m, J, N, max_chunk=64, with_grad=with_grad)))
    return out


def _check(runs, recs, thetas, kernel=S.SMC_KERNEL_RW, grads=None):
    for i, (w, m, _) in enumerate(runs):
        p1 = S.Population(m, w.J, w.N, max_chunk=64, with_grad=grads is not None)
        b = S.smc_run(m, p1, seed=SEEDS[i], Lmax=700, RmaxRec=64, kernel=kernel).summary()
        a = recs[i].summary()
        assert a["L"] == b["L"] and a["L"] > 1, i
        assert np.array_equal(a["t_end"], b["t_end"]) and np.array_equal(a["R"], b["R"]), i
        assert np.array_equal(a["n_accept"], b["n_accept"]), i
        assert np.array_equal(a["group_logwbar"], b["group_logwbar"]), i
        assert a["log_ml"] == b["log_ml"] and a["nse"] == b["nse"], i
        assert a["evals"] == b["evals"] and a["mh_steps"] == b["mh_steps"], i
        assert torch.equal(thetas[i], p1.theta), i
        if grads is not None:
            assert torch.equal(grads[i], p1.grad), i


@pytest.mark.parametrize("kernel", [S.SMC_KERNEL_RW, S.SMC_KERNEL_MALA])
@pytest.mark.parametrize("prec", [S.SMC_FP64, S.SMC_FP32])
def test_batch_of_ten_equals_single_runs(prec, kernel):
    mala = kernel == S.SMC_KERNEL_MALA
    runs = _runs(prec, with_grad=mala)
    recs = S.smc_run_batch([m for _, m, _ in runs], [p for _, _, p in runs], SEEDS, Lmax=700,
                           RmaxRec=64, kernel=kernel)
    torch.cuda.synchronize()
    _check(runs, recs, [p.theta for _, _, p in runs], kernel,
           [p.grad for _, _, p in runs] if mala else None)


def test_batch_on_a_side_stream():
    """The outputs are read on the caller's stream, which has every lane
    behind it when the call returns, with no device synchronisation."""
    runs = _runs(S.SMC_FP32)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        recs = S.smc_run_batch([m for _, m, _ in runs], [p for _, _, p in runs], SEEDS, Lmax=700,
                               RmaxRec=64)
        thetas = [p.theta.clone() for _, _, p in runs]
        weights = [r.group_logwbar.clone() for r in recs]
    side.synchronize()
    for r, x in zip(recs, weights):
        assert torch.equal(r.group_logwbar, x)
    _check(runs, recs, thetas)


@pytest.mark.parametrize("shape", [(128, 16), (256, 4)])
def test_batch_of_ten_in_any_shape_is_the_same_batch(shape):
    res = {}
    for sh in ((64, 8), shape):
        runs = _runs(S.SMC_FP32, shape=sh)
        recs = S.smc_run_batch([m for _, m, _ in runs], [p for _, _, p in runs], SEEDS, waves=7,
                               Lmax=700, RmaxRec=64)
        res[sh] = ([r.summary() for r in recs], [theta_np(p) for _, _, p in runs])
    for (a, tha), (b, thb) in zip(zip(*res[(64, 8)]), zip(*res[shape])):
        assert np.array_equal(a["n_accept"], b["n_accept"])
        assert a["log_ml"] == b["log_ml"]
        assert np.array_equal(tha, thb)
