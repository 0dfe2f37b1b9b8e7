"""Direct-act lists of more than 7,680 entries (a big leaf beside a clump of
thousands of leaves), which the whole chip orders and splits entry by entry:
psi and alpha against the oracle's direct sum, the work against Algorithm 1's
lists, and the same sums from a plan whose other targets are gone."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies
from parity_util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [(0, 1e-10), (1, 1e-6)], ids=["fp64", "fp32-mixed"])
@pytest.mark.parametrize("clumps,n,leaf", [(1, 9000, 1), (1, 60000, 4), (3, 40000, 2), (2, 100000, 16)])
def test_huge_lists(clumps, n, leaf, precision, tol, oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(270 + clumps)
    centre = skies.uniform(clumps, rng)
    p = np.repeat(centre, n, axis=1) + 2e-3 * rng.standard_normal((3, clumps * n))
    src = np.ascontiguousarray(np.concatenate([p / np.linalg.norm(p, axis=0), skies.uniform(40, rng)], axis=1))
    q = skies.masses_lognormal(src.shape[1], rng)
    near = np.repeat(centre, 60, axis=1) + 0.3 * rng.standard_normal((3, 60 * clumps))
    tgt = np.concatenate([near / np.linalg.norm(near, axis=0), skies.uniform(100, rng)], axis=1)
    opt = dict(tolerance=tol, leaf_size=leaf, precision=precision)
    out = []
    for t in (tgt, np.ascontiguousarray(tgt[:, : 30 * clumps])):
        plan = sf.Plan(src, q, t, **opt)
        psi, defl = plan.execute()
        torch.cuda.synchronize()
        w, (_, p2p) = plan.export_work(), plan.export_lists()
        per = np.bincount(p2p[:, 1], minlength=w["tgt_count"].size)[w["tgt_count"] > 0]
        print(f"[huge] {clumps} clumps: {(per > 7680).sum()} lists beyond 7,680, longest {per.max()}", flush=True)
        assert (per > 7680).sum() >= 1
        # every entry is summed or taken through its expansion, once
        cnt, t = plan.export_boxes()["count"], w["tgt_count"]
        held = np.flatnonzero(t > 0)
        assert np.array_equal(w["evals"][held] // t[held] <= per, np.ones(held.size, bool))
        if leaf == 1:
            assert np.array_equal(w["pairs"][held] // t[held] + w["evals"][held] // t[held], per)
        out.append((psi.cpu().numpy(), defl.cpu().numpy(), plan.export_keys()))
        plan.close()
    (psi, defl, keys), (psi2, defl2, _) = out
    rp, ra = oracle.direct(src, q, tgt)
    check(f"huge lists {clumps} x {n}", psi, defl, rp, ra, tol)
    # leaves that lost no target: the same list, the same sums
    m2 = psi2.size
    leaf_of = np.empty(tgt.shape[1], np.int64)
    leaf_of[keys["tgt_perm"]] = keys["tgt_leaf"]
    same = ~np.isin(leaf_of[:m2], leaf_of[m2:])
    assert np.abs(psi[:m2] - psi2)[same].max(initial=0) <= 1e-12 * np.abs(psi).max()
    assert np.abs(defl[:, :m2] - defl2)[:, same].max(initial=0) <= 1e-12 * np.abs(defl).max()
