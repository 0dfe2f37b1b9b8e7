"""sfmm_plan_info: a plan's own sizes without Algorithm 1's full lists."""
import numpy as np
import pytest

from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu
LISTS = ("n_m2l", "n_p2p", "m2l_order_sq")


def _sky(seed, n=20000, every=101):
    rng = skies.rng_for(seed)
    src = skies.clustered(n, rng, n_clumps=30)
    return src, skies.masses_lognormal(n, rng), np.ascontiguousarray(src[:, ::every])


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("n", [0, 300, 20000])
def test_info_is_the_statistics_without_the_lists(n, policy):
    """Before an execute and after each of two: the other fields agree, and the
    sum of the squared orders is the same at every request."""
    import paper_2210_07021_amd as sf
    src, q, tgt = _sky(210, n) if n else (np.zeros((3, 0)), np.zeros(0), skies.uniform(50, skies.rng_for(210)))
    plan = sf.Plan(src, q, tgt, tolerance=1e-6, leaf_size=8, order_policy=policy)
    sums = []
    for k in range(3):
        info, st = plan.info(), plan.stats()
        assert all(info[f] == -1 for f in LISTS)
        assert {f: v for f, v in info.items() if f not in LISTS} == {f: v for f, v in st.items() if f not in LISTS}
        assert info["n_leaves"] == (plan.export_boxes()["child0"] < 0).sum()
        sums.append(st["m2l_order_sq"])
        plan.execute()
    st = plan.stats()
    assert sums[0] == 0 and sums[1] == sums[2] == st["m2l_order_sq"]
    if n == 20000:
        fixed = st["n_m2l"] * st["order"] ** 2
        assert st["fell_back"] == 0 and (0 < sums[1] < fixed if policy else sums[1] == fixed)
    plan.close()


def test_a_plan_whose_full_lists_do_not_fit(monkeypatch):
    """Few targets: the plan's own lists fit, Algorithm 1's over all boxes do not.
    What needs them is refused; the plan, its sizes and the other exports are not."""
    import paper_2210_07021_amd as sf
    sky = _sky(211, every=2001)
    plan = sf.Plan(*sky, order=12, leaf_size=8)
    ref = [x.cpu().numpy() for x in plan.execute()]
    st, boxes, work, mult = plan.stats(), plan.export_boxes(), plan.export_work(), plan.export_expansions()[0]
    plan.close()
    monkeypatch.setenv("SFMM_LIST_LIMIT", str(min(st["n_m2l"], st["n_p2p"]) - 1))
    plan = sf.Plan(*sky, order=12, leaf_size=8)
    for a, b in zip(ref, plan.execute()):
        assert np.array_equal(a, b.cpu().numpy())
    assert plan.info()["n_boxes"] == st["n_boxes"]
    for a, b in ((boxes, plan.export_boxes()), (work, plan.export_work())):
        assert all(np.array_equal(a[k], b[k]) for k in a)
    for call in (plan.stats, plan.export_lists, plan.export_expansions):
        with pytest.raises(sf.SfmmError, match="interaction lists too large") as e:
            call()
        assert e.value.status == sf.SFMM_ERR_INVALID_ARG
    monkeypatch.delenv("SFMM_LIST_LIMIT")
    assert plan.stats()["n_m2l"] == st["n_m2l"]
    assert np.array_equal(plan.export_expansions()[0], mult)
    plan.close()
