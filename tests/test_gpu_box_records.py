"""Box geometry by lane teams: the same number for number whether one lane or
eight make a box (trees up to 12,288 boxes: eight), and the oracle's radius."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


def test_box_geometry_either_way(oracle_lib):
    import paper_2210_07021_amd as sf
    rng = skies.rng_for(171)
    src = skies.clustered(40000, rng, n_clumps=40)
    q = skies.masses_lognormal(40000, rng)
    few, many = [sf.Plan(src, q, skies.grid(1), order=8, leaf_size=leaf) for leaf in (64, 4)]
    a, b = few.export_boxes(), many.export_boxes()
    few.close()
    many.close()
    assert len(a["level"]) <= 12288 < len(b["level"])
    at = {(int(l), int(p)): i for i, (l, p) in enumerate(zip(b["level"], b["pixel"]))}
    k = np.array([at[(int(l), int(p))] for l, p in zip(a["level"], a["pixel"])])
    assert np.array_equal(a["centre"], b["centre"][:, k])
    assert np.array_equal(a["radius"], b["radius"][k])
    for i in range(0, k.size, 97):
        assert a["radius"][i] == pytest.approx(oracle.box_radius(int(a["level"][i]), int(a["pixel"][i])), rel=1e-15)
