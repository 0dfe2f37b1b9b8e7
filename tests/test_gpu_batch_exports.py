"""Exports of a kept batch's plans while its graph works on them: they read the
plans and write nothing of theirs."""
import ctypes

import numpy as np
import pytest

from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tier", [False, True])
def test_exports_beside_replays(tier):
    """Few targets, so that most boxes' local expansions are made for the export
    alone; the replay on another stream keeps its own and gives the same bits."""
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(200)
    lib = sf.load_library()
    src = [skies.clustered(60000 + 1000 * i, rng, n_clumps=30) for i in range(3)]
    q = [skies.masses_lognormal(x.shape[1], rng) for x in src]
    tgt = [np.ascontiguousarray(x[:, :40]) for x in src]
    batch = sf.Batch(src, q, tgt, order=20, leaf_size=8, precision=sf.SFMM_FP32_MIXED if tier else sf.SFMM_FP64)
    stream = torch.cuda.Stream()
    psi = [torch.empty(40, dtype=torch.float64, device="cuda") for _ in src]
    defl = [torch.empty((3, 40), dtype=torch.float64, device="cuda") for _ in src]
    pp = (ctypes.c_void_p * 3)(*[x.data_ptr() for x in psi])
    dp = (ctypes.c_void_p * 3)(*[x.data_ptr() for x in defl])
    torch.cuda.synchronize()

    def run():
        assert lib.sfmm_batch_execute(batch._h, pp, dp, ctypes.c_void_p(stream.cuda_stream)) == 0

    for _ in range(2):  # direct, direct and recorded
        run()
    stream.synchronize()
    ref = [x.cpu().numpy() for x in psi + defl]
    plans = [batch.plan(i) for i in range(3)]
    held = [p.export_work()["tgt_count"] > 0 for p in plans]
    assert all(h.sum() <= 40 for h in held)
    quiet = [p.export_expansions() for p in plans]
    assert all((np.abs(loc).max(axis=1) > 0).sum() > 1000 for _, loc in quiet)
    for k in range(12):
        run()  # a replay
        mult, loc = plans[k % 3].export_expansions()
        stream.synchronize()
        assert np.array_equal(mult, quiet[k % 3][0]) and np.array_equal(loc, quiet[k % 3][1]), k
        for a, b in zip(ref, psi + defl):
            assert np.array_equal(a, b.cpu().numpy()), k
    batch.close()
