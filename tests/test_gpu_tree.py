"""The one-pass tree build (k_tree.hip) where it can go wrong: point counts
around its 64-point steps and 512-point tiles, leaf sizes down to 1, above a
tile and above N, duplicated points (the same key on both sides of a tile edge)
and a clump down to the deepest level.  Keys, order and box tables are compared
exactly with the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(63, 1), (64, 2), (65, 64), (511, 3), (512, 1), (513, 511), (513, 512), (1025, 600),
                                 (1537, 7), (2000, 2000), (2000, 1999), (4097, 33)])
@pytest.mark.parametrize("kind", ["uniform", "duplicates", "clump"])
def test_tree_matches_oracle(kind, n, m, oracle_lib):
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(150 + n)
    src = skies.uniform(n, rng)
    if kind == "duplicates":  # runs of equal points, up to a tile long, within the leaf size or not
        src = np.repeat(src, rng.integers(1, 9, n), axis=1)[:, :n]
        src[:, n // 3:n // 3 + min(m, n // 3)] = src[:, [n // 3]]
    if kind == "clump":
        d = rng.standard_normal((3, n // 2)) * 10.0 ** rng.uniform(-8, -2, n // 2)
        c = src[:, :1] + d
        src[:, :n // 2] = c / np.linalg.norm(c, axis=0)
    src = np.ascontiguousarray(src)
    ot = oracle.tree(src, m)
    plan = sf.Plan(src, np.ones(n), skies.grid(4), order=4, leaf_size=m)
    b = plan.export_boxes()
    for f in ("level", "pixel", "first", "count", "parent", "child0"):
        assert np.array_equal(b[f], getattr(ot, f)), f
    k = plan.export_keys()
    assert np.array_equal(k["src_keys"], ot.keys) and np.array_equal(k["src_perm"], ot.perm)
    plan.close()


@pytest.mark.parametrize("max_level", [0, 1, 2, 29])
def test_level_cap(max_level, oracle_lib):
    """Duplicated points (more than m of them) go down to the cap."""
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(151)
    src = np.repeat(skies.uniform(40, rng), 5, axis=1)
    plan = sf.Plan(src, np.ones(200), skies.grid(4), order=4, leaf_size=3, max_level=max_level)
    b = plan.export_boxes()
    plan.close()
    assert b["level"].max() == max_level
    leaf = b["child0"] < 0
    assert b["count"][leaf].sum() == 200
    assert (b["level"][leaf & (b["count"] > 3)] == max_level).all()
    split = ~leaf
    assert (b["count"][split] > 3).all()
    for q in range(4):
        assert np.array_equal(b["parent"][b["child0"][split] + q], np.flatnonzero(split))
