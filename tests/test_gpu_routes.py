"""Routes of an execute that other calls do not take: on a stream that the
caller captures (trees of five levels and more run on one stream there), a
batch's pass taken into the caller's graph before it has one of its own, a
batch's replays with an empty shell, outputs handed in again and again, and
charges that are not finite."""
import ctypes

import numpy as np
import pytest

from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


def _sky(seed, n, m):
    rng = skies.rng_for(seed)
    return skies.clustered(n, rng, n_clumps=20), skies.masses_lognormal(n, rng), skies.uniform(m, rng)


def _between():
    """Other work and a wait between two replays"""
    import torch
    x = torch.randn(1 << 18, device="cuda")
    assert np.isfinite((x * x).sum().item())


@pytest.mark.parametrize("tier", [False, True])
@pytest.mark.parametrize("hessian", [False, True])
def test_execute_on_a_captured_stream(hessian, tier):
    import torch
    import paper_2210_07021_amd as sf
    plan = sf.Plan(*_sky(220, 40000, 9001), order=20, leaf_size=16,
                   precision=sf.SFMM_FP32_MIXED if tier else sf.SFMM_FP64)
    assert plan.export_boxes()["level"].max() >= 4
    call = plan.execute_hessian if hessian else plan.execute
    out = call()
    torch.cuda.synchronize()
    ref = [x.clone() for x in out]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        call(*out)
    for rep in range(4):
        for x in out:
            x.fill_(float("nan"))
        _between()
        if rep % 2:  # an eager call of the same plan in between
            for a, b in zip(ref, call()):
                assert torch.equal(a, b)
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref, out):
            assert torch.equal(a, b), rep
    plan.close()


@pytest.mark.parametrize("shells", [1, 3])
def test_batch_pass_in_the_callers_graph(shells):
    """Captured after one direct call with the same outputs: the caller's graph
    takes the pass itself.  With other outputs it is refused."""
    import torch
    import paper_2210_07021_amd as sf
    lib = sf.load_library()
    sky = [_sky(221 + i, 8000 + 5000 * i, 700) for i in range(shells)]
    batch = sf.Batch([x[0] for x in sky], [x[1] for x in sky], [x[2] for x in sky], order=16, leaf_size=16)

    def outputs():
        psi = [torch.full((700,), float("nan"), dtype=torch.float64, device="cuda") for _ in sky]
        return psi, [torch.full((3, 700), float("nan"), dtype=torch.float64, device="cuda") for _ in sky]

    def run(psi, defl, stream):
        arr = lambda xs: (ctypes.c_void_p * shells)(*[x.data_ptr() for x in xs])
        return lib.sfmm_batch_execute(batch._h, arr(psi), arr(defl), ctypes.c_void_p(stream.cuda_stream))

    (psi, defl), (psi2, defl2) = outputs(), outputs()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert run(psi, defl, stream) == 0
    stream.synchronize()
    ref = [x.clone() for x in psi + defl]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        refused = run(psi2, defl2, stream)
        taken = run(psi, defl, stream)
    assert refused == sf.SFMM_ERR_INVALID_ARG and taken == 0
    for rep in range(3):
        for x in psi + defl:
            x.fill_(float("nan"))
        _between()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref, psi + defl):
            assert torch.equal(a, b), rep
    for rep in range(4):  # and the batch's own calls afterwards: direct, recorded, replays
        for x in psi + defl:
            x.fill_(float("nan"))
        torch.cuda.synchronize()
        assert run(psi, defl, stream) == 0
        stream.synchronize()
        for a, b in zip(ref, psi + defl):
            assert torch.equal(a, b), rep
    batch.close()


def test_replays_with_an_empty_shell():
    """The third call and later ones replay the graph, the empty shell's zeros among its nodes."""
    import torch
    import paper_2210_07021_amd as sf
    sky = [_sky(230, 9000, 500), (np.zeros((3, 0)), np.zeros(0), skies.uniform(333, skies.rng_for(231))),
           _sky(232, 3000, 400)]
    batch = sf.Batch([x[0] for x in sky], [x[1] for x in sky], [x[2] for x in sky], order=12, leaf_size=16)
    psi, defl = batch.execute()
    torch.cuda.synchronize()
    ref = [x.clone() for x in psi + defl]
    assert not psi[1].any().item() and not defl[1].any().item()
    for rep in range(5):
        for x in psi + defl:
            x.fill_(float("nan"))
        _between()
        batch.execute(psi, defl)
        torch.cuda.synchronize()
        for a, b in zip(ref, psi + defl):
            assert torch.equal(a, b), rep
    batch.close()


def test_outputs_handed_in_again():
    """The same output tensors, full of NaN, for every call: all of each is written."""
    import torch
    import paper_2210_07021_amd as sf
    plan = sf.Plan(*_sky(240, 30000, 7001), order=20, leaf_size=16)
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            out = plan.execute_hessian()
            ref = [x.clone() for x in out]
            for _ in range(4):
                for x in out:
                    x.fill_(float("nan"))
                plan.execute_hessian(*out)
                got = [x.clone() for x in out]
                for x in out:
                    x.fill_(float("inf"))
                stream.synchronize()
                for a, b in zip(ref, got):
                    assert torch.equal(a, b)
    plan.close()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_charges_that_are_not_finite(bad):
    """One such charge: its leaf's expansion and those of the boxes above it are
    not finite, all others are what they are without it, bit for bit (16 boxes go
    through the shifts of Lemma 2 side by side)."""
    import paper_2210_07021_amd as sf
    src, q, tgt = _sky(250, 20000, 400)
    mult = []
    for v in (q[777], bad):
        c = q.copy()
        c[777] = v
        plan = sf.Plan(src, c, tgt, order=18, leaf_size=16)
        psi, _ = plan.execute()
        boxes = plan.export_boxes()
        perm = plan.export_keys()["src_perm"]
        mult.append(plan.export_expansions()[0])
        finite = np.isfinite(psi.cpu().numpy())
        plan.close()
    assert not finite.any()
    at = int(np.flatnonzero(perm == 777)[0])
    holds = (boxes["first"] <= at) & (at < boxes["first"] + boxes["count"])
    assert 3 <= holds.sum() <= 30
    assert np.array_equal(mult[0][~holds], mult[1][~holds]) and not np.isfinite(mult[1][holds][:, 1]).any()
