"""Direct sums of leaves with few targets (one target a lane, workgroups that
take several items) and with more: both forms against the oracle's direct sum
and, for the targets that they share, against each other; leaves of one target
and of several groups of 64, targets on the sources themselves."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies
from parity_util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf,m", [(9000, 1, 7001), (60000, 2, 40003), (60000, 2, 100000)])
def test_few_targets_a_leaf(n, leaf, m, oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(410 + m % 7)
    src = skies.uniform(n, rng)
    q = skies.masses_lognormal(n, rng)
    centre = skies.uniform(1, rng)
    heap = centre + 1e-3 * rng.standard_normal((3, 900))  # more than a group of 64 in a leaf
    tgt = np.concatenate([heap / np.linalg.norm(heap, axis=0), src[:, :500], skies.uniform(m - 1400, rng)], axis=1)
    more = np.concatenate([tgt, skies.uniform(20 * n, rng)], axis=1)
    out = []
    for t, one in ((tgt, True), (more, False)):
        plan = sf.Plan(src, q, np.ascontiguousarray(t), tolerance=1e-10, leaf_size=leaf)
        psi, defl = plan.execute()
        torch.cuda.synchronize()
        leaves = plan.stats()["n_target_leaves"]
        assert leaves >= 4096 and (t.shape[1] <= 8 * leaves) == one
        out.append((psi.cpu().numpy()[:m], defl.cpu().numpy()[:, :m]))
        plan.close()
    pick = np.r_[0:1400, rng.integers(1400, m, 600)]
    rp, ra = oracle.direct(src, q, np.ascontiguousarray(tgt[:, pick]))
    for psi, defl in out:
        check(f"{n} sources, leaf {leaf}, {m} targets", psi[pick], defl[:, pick], rp, ra, 1e-10)
    # the order of the sums over a team's lanes differs, nothing else
    assert np.abs(out[0][0] - out[1][0]).max() <= 1e-12 * np.abs(out[0][0]).max()
    assert np.abs(out[0][1] - out[1][1]).max() <= 1e-12 * np.abs(out[0][1]).max()
