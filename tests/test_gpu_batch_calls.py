"""Which calls of a batch run directly, record and replay: every order of calls
with two sets of outputs gives the plans' own results, bit for bit."""
import numpy as np
import pytest

from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shells", [1, 2, 5])
@pytest.mark.parametrize("calls", ["aaaa", "abab", "aabbaab", "abbbaaa"])
def test_call_orders(shells, calls):
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(180)
    src = [skies.clustered(700 * (i + 1), rng, n_clumps=4) for i in range(shells)]
    q = [skies.masses_lognormal(x.shape[1], rng) for x in src]
    tgt = [skies.uniform(300 + i, rng) for i in range(shells)]
    ref = []
    for x in zip(src, q, tgt):
        plan = sf.Plan(*x, tolerance=1e-8, leaf_size=16)
        ref.append([o.cpu().numpy() for o in plan.execute()])
        plan.close()
    batch = sf.Batch(src, q, tgt, tolerance=1e-8, leaf_size=16)
    out = {}
    for k, c in enumerate(calls):
        if c not in out:
            out[c] = batch.execute()
        else:
            for x in out[c][0] + out[c][1]:
                x.fill_(float("nan"))
            torch.randn(1 << 16, device="cuda").sum().item()  # other work between the calls
            batch.execute(*out[c])
        torch.cuda.synchronize()
        for i, (p, a) in enumerate(ref):
            assert np.array_equal(out[c][0][i].cpu().numpy(), p), (k, i)
            assert np.array_equal(out[c][1][i].cpu().numpy(), a), (k, i)
    batch.close()
