"""The direct acts on a second stream beside Lemmas 2 to 4 (trees of five levels
and more) and all on one stream (while stages are timed): the same additions in
the same order, so the results are equal bit for bit, on the default stream
and others, with several threads at once, and with the outputs used and
overwritten on the caller's stream right before and after the call."""
import threading

import numpy as np
import pytest

from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


def _case(n, m, seed):
    rng = skies.rng_for(seed)
    return (skies.clustered(n, rng, n_clumps=20), skies.masses_lognormal(n, rng), skies.uniform(m, rng))


def _one_stream(sf, plan, hessian):
    import torch
    sf.profile_enable(True)
    try:
        out = plan.execute_hessian() if hessian else plan.execute()
        torch.cuda.synchronize()
    finally:
        sf.profile_enable(False)
    return [x.cpu().numpy() for x in out]


@pytest.mark.parametrize("tier", [False, True])
@pytest.mark.parametrize("hessian", [False, True])
@pytest.mark.parametrize("n,m", [(700, 300), (20000, 1), (60000, 30001)])
def test_same_bits(n, m, hessian, tier, oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    src, q, tgt = _case(n, m, 180)
    plan = sf.Plan(src, q, tgt, order=20, leaf_size=16, precision=sf.SFMM_FP32_MIXED if tier else sf.SFMM_FP64)
    assert plan.export_boxes()["level"].max() >= 4
    ref = _one_stream(sf, plan, hessian)
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            out = None
            for _ in range(4):
                if out is not None:
                    for x in out:
                        x.fill_(float("nan"))
                out = plan.execute_hessian() if hessian else plan.execute()
                got = [x.clone() for x in out]
            stream.synchronize()
        for a, b in zip(ref, got):
            assert np.array_equal(a, b.cpu().numpy())
    plan.close()


def test_threads(oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    cases = [_case(15000 + 3000 * k, 5000, 181 + k) for k in range(4)]
    plans = [sf.Plan(*c, order=20, leaf_size=16) for c in cases]
    ref = [_one_stream(sf, p, False) for p in plans]
    bad = []

    def work(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(5):
                out = plans[k].execute()
                stream.synchronize()
                if not all(np.array_equal(a, b.cpu().numpy()) for a, b in zip(ref[k], out)):
                    bad.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for p in plans:
        p.close()
    assert not bad
