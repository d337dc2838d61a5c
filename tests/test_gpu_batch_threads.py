"""Adaptive batches of several host threads at a time, a stream each, and of new
threads after them (each call borrows its streams and decision slots from a
store shared by the threads): every batch equals the same batch on its own."""
import threading

import pytest
import torch

import paper_1304_4334_amd as S
import synthdata as SD

pytestmark = pytest.mark.gpu

SPECS = [("egarch11", 400, 4, 64, 0), ("egarch2t", 250, 4, 96, 1), ("egarch11", 700, 2, 200, 2),
         ("egarch2t", 333, 8, 32, 3), ("egarch11", 90, 2, 1000, 4), ("egarch11", 395, 2, 65, 6)]
SEEDS = [71, 72, 73, 74, 75, 76]


def _batch():
    models, pops = [], []
    for name, T, J, N, off in SPECS:
        w = SD.workload(name, T=T, J=J, N=N, seed_offset=off)
        models.append(S.Model(w.kind, w.y[:T], K=w.K, shock=w.shock, precision=S.SMC_FP32))
        pops.append(S.Population(models[-1], J, N, max_chunk=64))
    return models, pops


def _run(models, pops):
    recs = S.smc_run_batch(models, pops, SEEDS, Lmax=700, RmaxRec=64)
    return [r.summary()["log_ml"] for r in recs], [p.theta.clone() for p in pops]


def test_batches_of_several_threads():
    want = _run(*_batch())
    work = [_batch() for _ in range(3)]
    torch.cuda.synchronize()
    for rep in range(3):
        out = [None] * 3

        def call(k):
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                out[k] = _run(*work[k])
            s.synchronize()

        threads = [threading.Thread(target=call, args=(k,)) for k in range(3)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for k in range(3):
            assert out[k] is not None and out[k][0] == want[0], (rep, k)
            assert all(torch.equal(a, b) for a, b in zip(out[k][1], want[1])), (rep, k)
