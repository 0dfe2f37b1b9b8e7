"""Segments and target groups of the expansions at targets.

Segment lengths by the number of target leaves (16 below 16,384 leaves, 64
below 65,536) and groups of 64 targets side by side where a leaf holds many:
the same terms in another order, so plans of different lengths agree to the
rounding of their sums (some thousand additions at a target, 1e-12 of the
field's rms) and with the direct sum at the tolerance, 1e-10."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tier", [False, True])
@pytest.mark.parametrize("n,leaf,m", [(3000, 16, 70), (3000, 32, 63), (20000, 32, 200001), (1500, 64, 150000),
                                      (60000, 2, 60000)])
def test_segment_lengths(n, leaf, m, tier, oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(170)
    src = skies.clustered(n, rng, n_clumps=5)
    q = skies.masses_lognormal(n, rng)
    tgt = skies.uniform(m, rng)
    got = []
    for seg in (0, 8, 4096):
        plan = sf.Plan(src, q, tgt, order=38, leaf_size=leaf, far_segment=seg,
                       precision=sf.SFMM_FP32_MIXED if tier else sf.SFMM_FP64)
        psi, defl, hess = plan.execute_hessian()
        torch.cuda.synchronize()
        got.append([x.cpu().numpy() for x in (psi, defl, hess)])
        plan.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.abs(a - b).max() <= 1e-12 * np.sqrt((a * a).mean()) + 1e-12 * np.abs(a).max()
    if not tier:
        k = np.arange(0, m, max(1, m // 300))
        ref_p, ref_a = oracle.direct(src, q, np.ascontiguousarray(tgt[:, k]))
        assert np.linalg.norm(got[0][0][k] - ref_p) < 1e-10 * np.linalg.norm(ref_p)
        assert np.linalg.norm(got[0][1][:, k] - ref_a) < 1e-10 * np.linalg.norm(ref_a)
