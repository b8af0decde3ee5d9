"""Which workgroup of a scheduled attention call takes which unit (sched_order, sched_position), through a small program
that includes their header: no GPU needed. The last of several rounds is given out by accumulated work, as the metadata
kernels do it."""
import os
import subprocess
from statistics import NormalDist

import pytest

from paper_2503_05096_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS, W = 256, 512
FIXED, BLOCK = 2, 32                # a unit's fixed work in token blocks, tokens per block


@pytest.fixture(scope="module")
def schedule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("sched") / "sched_driver")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", build.INCLUDE,
                           os.path.join(ROOT, "tests", "native", "sched_driver.cpp"), "-o", exe])

    def run(work, w=W, cus=CUS):
        """(order, units by position per round)"""
        text = " ".join(map(str, [w, cus, len(work), *work]))
        got = list(map(int, subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()))
        return got[0], [got[1 + r * w:1 + (r + 1) * w] for r in range((len(got) - 1) // w)]
    return run


def uniform(n, lo, hi):
    return sorted((-(-(lo + (hi - lo) * k // max(n - 1, 1)) // BLOCK) + FIXED for k in range(n)), reverse=True)


def lognormal(n, lo, hi):
    mid = 1.4 * (lo * hi) ** 0.5
    at = (NormalDist(0, 0.7).inv_cdf((k + 0.5) / n) for k in range(n))
    return sorted((-(-int(min(hi, max(lo, mid * 2.718281828 ** a))) // BLOCK) + FIXED for a in at), reverse=True)


def fullest(work, rounds):
    """work of the fullest compute unit over the mean, the last of several rounds by accumulated work"""
    cu = [0] * CUS
    plain = rounds[:-1] if len(rounds) > 1 else rounds
    for units in plain:
        for w, k in enumerate(units):
            cu[w % CUS] += work[k] if k < len(work) else 0
    for base in range(len(plain) * W, len(work), CUS):
        for k, c in zip(range(base, min(base + CUS, len(work))), sorted(range(CUS), key=cu.__getitem__)):
            cu[c] += work[k]
    return max(cu) / (sum(cu) / CUS)


@pytest.mark.parametrize("cus", [256, 120, 64])
@pytest.mark.parametrize("slots", [1, 2, 3, 4])
def test_every_unit_is_taken_once(schedule, slots, cus):
    w = slots * cus
    for width in (w, w - 1, w // 2 + 1):
        for total in (1, cus, cus + 1, width, width + 1, width + cus // 2, width + cus, width + cus + 1, 2 * width, 3 * width + 5, 5 * width):
            for work in (uniform(total, 40, 900), lognormal(total, 40, 2000)):
                _, rounds = schedule(work, width, cus)
                for r, units in enumerate(rounds):
                    assert sorted(units) == list(range(r * width, (r + 1) * width)), (width, total, r)


def test_one_round_is_even(schedule):
    assert fullest(uniform(512, 1024, 2048), schedule(uniform(512, 1024, 2048))[1]) <= 1.02
    work = lognormal(512, 128, 2000)
    assert fullest(work, schedule(work)[1]) < fullest(work, [list(range(W))])


@pytest.mark.parametrize("total", [513, 540, 600, 650, 700])
def test_a_few_third_units_do_not_go_on_top_of_even_totals(schedule, total):
    """Units about as long as each other: a third one on top of an even pair makes that compute unit half as long again."""
    for lo, hi in ((500, 1500), (1000, 1900)):
        work = uniform(total, lo, hi)
        order, rounds = schedule(work)
        assert order == total - W, (lo, hi)
        assert fullest(work, rounds) <= 1.1, (lo, hi, fullest(work, rounds))


def test_skewed_lengths_keep_even_pairs(schedule):
    """Pairs of the longest units would be far longer than any other compute unit's work."""
    for total in (540, 600, 700):
        work = lognormal(total, 128, 2000)
        order, rounds = schedule(work)
        assert order == 0 and fullest(work, rounds) <= 1.3, total
