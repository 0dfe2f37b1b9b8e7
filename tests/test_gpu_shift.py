"""Lemmas 2 and 4 on the matrix cores (k_shift.hip) against the lemmas as
printed (the oracle's triple sums): every remainder of the order by the tile
width 4, one tile and several, shallow trees (both shifts full) and a tree
down to level ~20, where one shift parameter of each lemma runs through the
banded and the identity forms.

Coefficients are compared in the box's own scale (A_l / rho^l for multipoles,
A_l rho^l for locals), each against the largest of its record.  Tolerance:
about 2 p additions a level of terms of that size, times the binomial growth
of a shift that the MACs keep below ~2^5: 1e-12 at the orders here, ten times
that for locals, which gather ~25 translations."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


def _local_coords(c, pts):
    """(theta, phi) of pts in the system of centre c from differences: the
    oracle's own form projects pts themselves, which at a distance of 1e-6
    leaves 1e-10 of the angles (the box centres are the same FP64 numbers on
    both sides, so this is the reference's rounding, not the method's)."""
    from oracle import lemmas as L
    e_t, e_p, _ = L.frame(c)
    pts = np.asarray(pts, dtype=np.float64).reshape(3, -1)
    c = np.asarray(c, dtype=np.float64).reshape(3, 1)
    d, s = pts - c, pts + c
    theta = 2.0 * np.arctan2(np.sqrt((d * d).sum(0)), np.sqrt((s * s).sum(0)))
    return theta, np.arctan2(e_p @ d, e_t @ d)


def _sky(kind):
    rng = skies.rng_for(140)
    src = skies.uniform(300, rng)
    if kind == "deep":
        c = skies.uniform(2, rng)
        d = rng.standard_normal((3, 120)) * np.repeat([1e-6, 3e-5], 60)
        p = np.repeat(c, 60, axis=1) + d
        src = np.concatenate([src[:, :150], p / np.linalg.norm(p, axis=0)], axis=1)
    q = skies.masses_lognormal(src.shape[1], rng)
    tgt = np.concatenate([src[:, ::3], skies.uniform(40, rng)], axis=1)
    return src, q, tgt


@pytest.mark.parametrize("kind", ["shallow", "deep"])
@pytest.mark.parametrize("order", [1, 2, 3, 4, 5, 7, 8, 10, 13])
def test_up_and_down_passes_match_lemmas(kind, order, oracle_lib, monkeypatch):
    import torch
    import paper_2210_07021_amd as sf
    from oracle import lemmas as L
    monkeypatch.setattr(L, "local_coords", _local_coords)
    src, q, tgt = _sky(kind)
    plan = sf.Plan(src, q, tgt, order=order, leaf_size=4)
    plan.execute()
    torch.cuda.synchronize()
    mult, loc = plan.export_expansions()
    plan.close()
    ref = L.sfmm(src, q, tgt[:, :1], p=order, m=4)
    ot = ref["tree"]
    l = np.arange(1, order + 1)
    worst = {"m": 0.0, "l": 0.0}
    for bx in range(ot.nbox):
        rho = np.tan(ot.radius[bx] / 2.0)
        for got, (C, Q, A), kind_ in ((mult[bx], ref["multipole"][bx], "m"), (loc[bx], ref["local"][bx], "l")):
            if not np.ndim(A) or (kind_ == "m" and ot.count[bx] == 0):
                continue
            f = rho ** l if kind_ == "l" else rho ** -l.astype(float)
            e = np.concatenate([[C, Q], A * f])
            g = np.concatenate([got[:2], (got[2::2] + 1j * got[3::2]) * f])
            worst[kind_] = max(worst[kind_], np.abs(g - e).max() / max(np.abs(e).max(), 1e-300))
    print(f"[shift] {kind} p={order}: levels {ot.level.max() + 1}, worst scaled coefficient error multipole "
          f"{worst['m']:.2e} local {worst['l']:.2e}", flush=True)
    assert worst["m"] < 1e-12 and worst["l"] < 1e-11
