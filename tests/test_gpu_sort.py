"""The key sorts (k_sort.hip, and the radix sort above and beside them) seen
through a plan's source keys and permutation: NumPy's stable sort is the
reference, and everything is equal bit for bit.

Sizes lie at the edges of a wave, a workgroup, what one workgroup sorts
(8,192), the bucket numbers' steps (65,536 and 1,048,576 keys) and the largest
sampled sort (10,485,760).  Orders: random; sorted and reversed; coincident
points in runs below and above a bucket; clumps tighter than the 32 bits of the
first window; and one that hides a clump from every sampled position, whose
bucket is then larger than a workgroup's memory."""
import numpy as np
import pytest

import oracle
from paper_2210_07021_amd import skies

pytestmark = pytest.mark.gpu


def _clump(n, width, rng):
    c = skies.uniform(1, rng)
    p = c + width * rng.standard_normal((3, n))
    return p / np.linalg.norm(p, axis=0)


def _check(src, m=64):
    import paper_2210_07021_amd as sf
    n = src.shape[1]
    plan = sf.Plan(np.ascontiguousarray(src), np.ones(n), skies.grid(2), order=4, leaf_size=m)
    k = plan.export_keys()
    plan.close()
    keys = oracle.keys(src)
    perm = np.argsort(keys, kind="stable")
    assert np.array_equal(k["src_keys"], keys[perm]) and np.array_equal(k["src_perm"], perm)


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 16385, 65536, 65537, 131073])
def test_sizes(n, oracle_lib):
    _check(skies.uniform(n, skies.rng_for(170 + n)))


@pytest.mark.parametrize("n", [1 << 20, (1 << 21) + 1, 10 << 20, (10 << 20) + 1])
def test_large(n, oracle_lib):
    rng = skies.rng_for(171)
    _check(np.concatenate([skies.uniform(n // 2, rng), skies.clustered(n - n // 2, rng, n_clumps=40)], axis=1))


@pytest.mark.parametrize("n", [3000, 8192, 40000, 300000])
@pytest.mark.parametrize("kind", ["sorted", "reversed", "equal", "runs", "coincident", "clump", "clumps"])
def test_orders(kind, n, oracle_lib):
    rng = skies.rng_for(172)
    src = skies.uniform(n, rng)
    if kind in ("sorted", "reversed"):
        src = src[:, np.argsort(oracle.keys(src))]
        src = src if kind == "sorted" else src[:, ::-1]
    elif kind == "equal":
        src = np.repeat(src[:, :1], n, axis=1)
    elif kind == "runs":
        src = np.repeat(src, rng.integers(1, 40, n), axis=1)[:, :n][:, rng.permutation(n)]
    elif kind == "coincident":  # half of all points at one place, a tenth at another
        src[:, : n // 2] = src[:, :1]
        src[:, n // 2: n // 2 + n // 10] = src[:, -1:]
        src = src[:, rng.permutation(n)]
    elif kind == "clump":
        src[:, : n // 2] = _clump(n // 2, 1e-7, rng)
        src = src[:, rng.permutation(n)]
    else:
        for i in range(20):
            a, b = i * n // 40, (i + 1) * n // 40
            src[:, a:b] = _clump(b - a, 10.0 ** -(3 + i % 6), rng)
        src = src[:, rng.permutation(n)]
    _check(src)


def _sampled(n, ns):
    i = np.arange(ns, dtype=np.uint64)
    z = (i + np.uint64(1)) * np.uint64(0x9e3779b97f4a7c15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xbf58476d1ce4e5b9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94d049bb133111eb)
    z ^= z >> np.uint64(31)
    j = np.arange(ns + 1, dtype=np.int64) * n // ns
    return j[:-1] + ((z >> np.uint64(32)) * (j[1:] - j[:-1]).astype(np.uint64) >> np.uint64(32)).astype(np.int64)


@pytest.mark.parametrize("n", [40000, 300000])
def test_unsampled_clump(n, oracle_lib):
    rng = skies.rng_for(173)
    src = _clump(n, 1e-5, rng)
    src[:, ::7] = src[:, [0]]  # with equal keys among them
    nb = 16
    while nb * 4096 < n:
        nb *= 2
    at = _sampled(n, 16 * nb)
    src[:, at] = skies.uniform(at.size, rng)
    _check(src)
