"""The plan's pruned interaction lists (k_lists.hip): few and clustered targets
(most boxes without any), direct-act lists across the sizes where the ordering
changes its method (64, 256, 1024, 7680 entries: a sparse leaf next to a clump
of thousands of leaves), and looser MACs, whose hand-down lists outgrow their
room.  psi and alpha against the oracle's direct sum at the repository's gates;
the pruned work against Algorithm 1's full lists; and a target's result does
not depend on which other leaves hold targets."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies
from parity_util import check

pytestmark = pytest.mark.gpu


def _clump(n, width, rng, extra):
    c = skies.uniform(1, rng)
    p = c + width * rng.standard_normal((3, n))
    src = np.concatenate([p / np.linalg.norm(p, axis=0), skies.uniform(extra, rng)], axis=1)
    return np.ascontiguousarray(src), c


def _run(src, q, tgt, **opt):
    import torch
    import paper_2210_07021_amd as sf
    plan = sf.Plan(src, q, tgt, **opt)
    psi, defl = plan.execute()
    torch.cuda.synchronize()
    return plan, psi.cpu().numpy(), defl.cpu().numpy()


@pytest.mark.parametrize("precision,tol", [(0, 1e-10), (1, 1e-6)], ids=["fp64", "fp32-mixed"])
@pytest.mark.parametrize("n", [40, 150, 700, 3000, 12000])
def test_long_direct_lists(n, precision, tol, oracle_lib):
    """leaf size 1: a sparse leaf beside the clump sums every one of its
    leaves directly (the longest list is printed)."""
    rng = skies.rng_for(160)
    src, c = _clump(n, 2e-3, rng, 30)
    q = skies.masses_lognormal(src.shape[1], rng)
    near = c + 0.3 * rng.standard_normal((3, 40))
    tgt = np.concatenate([near / np.linalg.norm(near, axis=0), src[:, ::17], skies.uniform(50, rng)], axis=1)
    plan, psi, defl = _run(src, q, tgt, tolerance=tol, leaf_size=1, precision=precision)
    _, p2p = plan.export_lists()
    w = plan.export_work()
    held = np.flatnonzero(w["tgt_count"] > 0)
    per = np.bincount(p2p[:, 1], minlength=w["tgt_count"].size)[held]
    # every direct act of a leaf with targets is summed or taken through an
    # expansion: one particle a leaf here
    cnt = plan.export_boxes()["count"]
    assert (cnt[p2p[:, 0]] == 1).all()
    t = w["tgt_count"][held]
    assert np.array_equal(w["pairs"][held] // t + w["evals"][held] // t, per)
    assert (w["pairs"][w["tgt_count"] == 0] == 0).all()
    plan.close()
    rp, ra = oracle.direct(src, q, tgt)
    check(f"lists n={n} precision {precision} longest {per.max()}", psi, defl, rp, ra, tol)


@pytest.mark.parametrize("m", [1, 3, 65])
def test_few_targets(m, oracle_lib):
    """Targets in a handful of leaves: the same values as among many targets
    (the leaves, and so the near-field split, hold the same ones)."""
    rng = skies.rng_for(161)
    src = skies.clustered(20000, rng, n_clumps=40)
    q = skies.masses_lognormal(20000, rng)
    some = src[:, :m] if m > 1 else skies.uniform(1, rng)
    plan, psi, defl = _run(src, q, some, tolerance=1e-10, leaf_size=24)
    leaf = np.unique(plan.export_keys()["tgt_leaf"])
    full, _ = plan.export_lists()
    assert plan.stats()["n_m2l"] == full.shape[0]
    plan.close()
    rp, ra = oracle.direct(src, q, some)
    check(f"few targets {m} in {leaf.size} leaves", psi, defl, rp, ra, 1e-10)
    more = skies.uniform(3000, rng)
    plan, psi2, defl2 = _run(src, q, np.concatenate([some, more], axis=1), tolerance=1e-10, leaf_size=24)
    k = plan.export_keys()
    lf = np.empty(m + 3000, np.int64)
    lf[k["tgt_perm"]] = k["tgt_leaf"]
    alone = ~np.isin(lf[:m], lf[m:])  # leaves that got no other target
    assert np.abs(psi2[:m] - psi)[alone].max(initial=0) <= 1e-12 * np.abs(psi).max()
    assert np.abs(defl2[:, :m] - defl)[:, alone].max(initial=0) <= 1e-12 * np.abs(defl).max()
    plan.close()


@pytest.mark.parametrize("c_s,c_t", [(5.0, 0.2), (12.0, 0.08)])
def test_loose_macs(c_s, c_t, oracle_lib):
    """Hand-down lists of hundreds to thousands of sources (made again with
    exact sizes): the full method still gives the direct sum."""
    rng = skies.rng_for(162)
    src = skies.clustered(30000, rng, n_clumps=50)
    q = skies.masses_lognormal(30000, rng)
    tgt = np.concatenate([skies.grid(16), src[:, :300]], axis=1)
    plan, psi, defl = _run(src, q, tgt, tolerance=1e-10, leaf_size=8, c_s=c_s, c_t=c_t)
    plan.close()
    rp, ra = oracle.direct(src, q, tgt)
    check(f"loose MACs {c_s} {c_t}", psi, defl, rp, ra, 1e-10)
