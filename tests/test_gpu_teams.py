"""The lane teams of Lemmas 1 and 3 and of the direct sums on either side of
the sizes at which their widths change (Lemma 1: 16 lanes a leaf up to 131,072
boxes, four above; Lemma 3: 64 lanes a box up to 6,144 boxes, 16 up to 81,920,
two above; direct sums: four waves an item up to 4,096 items), with leaves of
every size by the quad and the row.

Lemma 1 against its sums in NumPy, each coefficient in the box's own scale and
against the sum of its terms' sizes: ~70 roundings of a term, 1e-13.  Fields
against the direct sum at 1e-10, the tolerance the orders are chosen for."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


def _sky(n, rng):
    """Half a uniform sky, half clumps of 1 .. 70 points tighter than any leaf"""
    k = np.arange(n // 2)
    sizes = 1 + np.arange(n) % 70
    owner = np.repeat(np.arange(n), sizes)[: n // 2]
    c = skies.uniform(int(owner[-1]) + 1, rng)[:, owner] + 1e-9 * rng.standard_normal((3, k.size))
    return np.ascontiguousarray(np.concatenate([skies.uniform(n - k.size, rng), c / np.linalg.norm(c, axis=0)], axis=1))


@pytest.mark.parametrize("order", [1, 2, 3, 4, 5, 38])
@pytest.mark.parametrize("n,leaf", [(3000, 70), (30000, 70), (160000, 1)])
def test_leaf_expansions(n, leaf, order, oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    from oracle import lemmas as L
    rng = skies.rng_for(160)
    src = _sky(n, rng)
    q = skies.masses_lognormal(n, rng)
    plan = sf.Plan(src, q, skies.grid(2), order=order, leaf_size=leaf, max_level=7)
    plan.execute()
    torch.cuda.synchronize()
    mult, _ = plan.export_expansions()
    b, perm = plan.export_boxes(), plan.export_keys()["src_perm"]
    plan.close()
    assert (len(b["level"]) > 131072) == (n > 100000)
    leaves = np.flatnonzero(b["child0"] < 0)
    worst, rho_min = 0.0, 1.0
    for bx in leaves[:: max(1, leaves.size // 400)]:
        cnt = int(b["count"][bx])
        if cnt == 0:
            assert not mult[bx].any()
            continue
        ids = perm[b["first"][bx]: b["first"][bx] + cnt]
        c = oracle.pix_point(int(b["level"][bx]), int(b["pixel"][bx]))
        rho = np.tan(oracle.box_radius(int(b["level"][bx]), int(b["pixel"][bx])) / 2.0)
        e_t, e_p, _ = L.frame(c)
        pts, d = src[:, ids], src[:, ids] - c[:, None]
        opc = 1.0 + c @ pts
        z = (e_t @ d + 1j * (e_p @ d)) / opc / rho
        qi = q[ids] / (4.0 * np.pi)
        Q = qi.sum()
        C = (qi * np.log(0.5 * opc)).sum() - Q * np.log(2.0)
        worst = max(worst, abs(mult[bx][0] - C) / Q, abs(mult[bx][1] - Q) / Q)
        for l in range(1, order + 1):
            A = -(qi * z ** l).sum() / l
            g = mult[bx][2 * l] + 1j * mult[bx][2 * l + 1]
            worst = max(worst, abs(g / rho ** l - A) / ((qi * np.abs(z) ** l).sum() / l))
        rho_min = min(rho_min, rho)
    bound = 8 * 2.0 ** -53 * (10 + order / rho_min)
    print(f"[teams] n={n} p={order}: worst {worst:.2e} bound {bound:.2e}", flush=True)
    assert worst < bound


@pytest.mark.parametrize("n,leaf,m", [(300, 64, 64), (1500, 4, 65), (20000, 4, 1), (20000, 64, 63), (150000, 2, 127)])
def test_fields(n, leaf, m, oracle_lib):
    import torch
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(161)
    src = skies.clustered(n, rng, n_clumps=max(4, n // 500))
    q = skies.masses_lognormal(n, rng)
    # targets at every source, so that most boxes have lists; those checked
    # lie in front of them
    check = np.concatenate([src[:, :: max(1, n // 100)], skies.uniform(m, rng)], axis=1)
    tgt = np.ascontiguousarray(np.concatenate([check, src], axis=1))
    plan = sf.Plan(src, q, tgt, tolerance=1e-10, leaf_size=leaf)
    psi, defl = plan.execute()
    torch.cuda.synchronize()
    psi, defl = psi.cpu().numpy(), defl.cpu().numpy()
    plan.close()
    k = check.shape[1]
    ref_p, ref_a = oracle.direct(src, q, np.ascontiguousarray(check))
    ep = np.linalg.norm(psi[:k] - ref_p) / np.linalg.norm(ref_p)
    ea = np.linalg.norm(defl[:, :k] - ref_a) / np.linalg.norm(ref_a)
    print(f"[teams] n={n} leaf={leaf}: psi {ep:.2e} deflection {ea:.2e}", flush=True)
    assert ep < 1e-10 and ea < 1e-10
