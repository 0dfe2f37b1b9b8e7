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


@pytest.mark.parametrize("tier", [False, True])
def test_no_allocation_scratch(tier, oracle_lib):
    """Short segments never take a plan beyond the no-allocation scratch (64 MB
    of partial slots at most), and that entry gives the same bits."""
    import ctypes
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(172)
    src = skies.clustered(300000, rng)
    q = skies.masses_lognormal(300000, rng)
    tgt = torch.from_numpy(skies.uniform(1000000, rng)).cuda()
    kw = dict(order=20, leaf_size=30, precision=sf.SFMM_FP32_MIXED if tier else sf.SFMM_FP64)
    plan = sf.Plan(src, q, tgt, **kw)
    long = sf.Plan(src, q, tgt, far_segment=128, **kw)
    short, most = plan.stats()["execute_scratch_bytes"], long.stats()["execute_scratch_bytes"]
    print(f"[segments] scratch {short} (segments of 128: {most})", flush=True)
    assert most <= 256 << 20 and short <= 256 << 20 and short <= max(most, 65 << 20) + 8 * 20 * 10**6
    psi, defl = plan.execute()
    p2, d2 = torch.empty_like(psi), torch.empty_like(defl)
    lib = sf.load_library()
    assert lib.sfmm_execute_noalloc(plan._h, ctypes.c_void_p(p2.data_ptr()), ctypes.c_void_p(d2.data_ptr()),
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    assert torch.equal(psi, p2) and torch.equal(defl, d2)
    plan.close()
    long.close()
