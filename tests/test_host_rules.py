"""Rules of the library compiled for the host (tests/host_rules.cpp, the same
headers as the HIP code)."""
import math
import os
import random
import re
import shutil
import subprocess
from decimal import Decimal, getcontext

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def host_rules(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("host_rules") / "host_rules")
    cmd = [HIPCC, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           os.path.join(HERE, "host_rules.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def _run(exe, mode, text=""):
    r = subprocess.run([exe, mode], input=text, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout.split("\n")


@pytest.mark.parametrize("total", [0, 5, 2**31 - 1, 2**31, 2**32 - 1, 2**32, 2**32 + 5, 3 * 2**32 + 7])
def test_list_totals_do_not_wrap(host_rules, total):
    """The totals of an interaction list, from per-box counts of up to 2^30: exact
    up to 2^32 - 1, which is as far as a refusal needs them, and never less
    than that beyond (a wrapped total of 2^32 + 5 entries read as 5)."""
    rng = random.Random(total)
    left, counts = total, [0]
    while left > 0:
        c = min(left, rng.choice([rng.randint(1, 1000), rng.randint(1, 2**30), 2**30]) if total > 10**6 else 1)
        counts.append(c)
        left -= c
    rng.shuffle(counts)
    got = [int(x) for x in _run(host_rules, "sums", " ".join(map(str, counts)) + "\n")[0].split()]
    assert got == [min(total, 2**32 - 1)] * 3


def test_walk_stack_stays_in_bounds(host_rules):
    """The stack of the list walk (LDS): no step from any state leaves it fewer
    than the spare places, except the depth-first ones that the spare is for, and
    those stay within it to the deepest level.  (One wave with 768 of 1,024
    places taken took 64 items, which left 64 places for up to 87.)"""
    for line in _run(host_rules, "stack"):
        if line:
            waves, states, bad, most, stack = (int(x) for x in line.split())
            assert states > 4000 * waves and bad == 0 and most <= stack, line


# Errors (log: largest, root mean square; reciprocal: the same) of the pair loop
# with the 128-entry table, the degree-7 series and a reciprocal refined by two
# Newton steps, measured over the same arguments: what holds must not be worse.
# (The largest of 2e6 varies with the table's own errors: 1 % room.)
PAIR_ERRORS = [(2.292e-16, 5.31e-17, 1.111e-16, 4.90e-17), (2.266e-16, 4.79e-17, 1.111e-16, 4.72e-17),
               (1.346e-16, 3.79e-17, 1.111e-16, 4.92e-17)]


def test_pair_log_and_reciprocal_keep_their_accuracy(host_rules):
    lines = _run(host_rules, "logerr")
    for line, was in zip(lines, PAIR_ERRORS):
        now = [float(x) for x in line.split()]
        assert all(a <= 1.01 * b for a, b in zip(now, was)), (now, was)


def test_pair_log_of_subnormal_arguments(host_rules):
    """|d|^2 below 2.2e-308 is a subnormal number: its mantissa, not its own bits,
    picks the table entry.  (The reciprocal is finite down to 5.6e-309.)"""
    rng = random.Random(5)
    xs = [10 ** rng.uniform(-323, -307) for _ in range(2000)] + [5e-324, 2.0**-1022, 2.0**-1022 - 2.0**-1074]
    for x, line in zip(xs, _run(host_rules, "log", "".join(x.hex() + "\n" for x in xs))):
        lg, inv = (float.fromhex(t) for t in line.split())
        assert abs(lg - math.log(x)) <= 2.5e-16 * abs(math.log(x)), x
        assert inv == math.inf or abs(inv * x - 1.0) <= 4 * 2.0**-52, x


def test_no_exception_leaves_a_c_entry():
    """Every C entry that can throw turns the library's errors and those of the
    standard library (no host memory for a copy) into a status."""
    text = open(os.path.join(HERE, "..", "paper_2210_07021_amd", "csrc", "sfmm_api.hip")).read()
    entries = re.split(r"\n(?=sfmm_status sfmm_|void sfmm_|const char\* sfmm_|int32_t sfmm_)", text[text.index('extern "C"'):])
    tried = [e for e in entries if re.search(r"\n    try \{", e)]
    assert len(tried) >= 19
    for e in tried:
        assert re.search(r"\n    \} catch \(const Error& e\) \{\n.*\n    \} catch \(const std::exception& e\) \{", e), e[:60]


def test_sort_keys_of_ordered_lists(host_rules):
    """The precision tier's direct acts are ordered by (round, first particle); a
    list's place below that key or a list's number above it has room of its own.
    (26 bits for the place once ran into the first particle in lists of 2^26.)"""
    rng = random.Random(9)
    firsts = sorted({rng.randrange(2**31) for _ in range(300)} | {0, 1, 2**31 - 1})
    rows = [(r, f, rng.choice([0, 7679, 2**26, 2**27 - 1, rng.randrange(2**27)])) for r in (2, 31, 32, 61) for f in firsts]
    out = _run(host_rules, "actkey", "".join("%d %d %d\n" % r for r in rows))
    for (_, _, e), line in zip(rows, out):
        assert [int(x) for x in line.split()] == [e, 1]
    # a list of more than 7,680 entries each: fewer than 2^31 / 7681 of them
    bits, fits = (int(x) for x in out[len(rows)].split())
    assert 2**bits > 2**31 // 7681 and fits == 1


def test_log_table_is_correctly_rounded(host_rules):
    getcontext().prec = 50
    for j, line in enumerate(_run(host_rules, "logtab")[:-1]):
        ci, nl = (float.fromhex(t) for t in line.split())
        assert ci == 1.0 / (0.5 + (j + 0.5) / 1024)
        assert nl == float(-Decimal(ci).ln()), j
    assert j == 511
