"""The rule by which the hard-sphere kernels skip blocks of beads
(real_skip.hpp), compiled for the host: never more steps than the exact
distance allows, over all bond lengths a call may have, and no fewer than
about one less in the ordinary range.
"""
import math
import os
import random
import subprocess
from fractions import Fraction

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1704_04381_amd", "csrc")


@pytest.fixture(scope="module")
def skip(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("skip") / "skip_rule")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, "-o", exe,
                           os.path.join(HERE, "pins", "skip_rule.cpp")])

    def run(cases):
        text = "\n".join(" ".join(float(v).hex() for v in c) for c in cases)
        return [int(v) for v in subprocess.check_output([exe], input=text, text=True).split()]
    return run


def _cases(exponents, n, seed):
    rng = random.Random(seed)
    cases = []
    for e in exponents:
        for _ in range(n):
            b = rng.uniform(1.0, 10.0) * 10.0 ** e
            sigma = b * rng.choice([0.0, 1e-6, 0.3, 0.75, 1.0, 1.9])
            d = b * rng.choice([rng.uniform(0.0, 4.0), rng.uniform(1.0, 40.0), math.exp(rng.uniform(0.0, 9.7))])
            cases.append((b, sigma, d))
    return cases


def test_never_more_steps_than_the_distance_allows(skip):
    cases = _cases(list(range(-165, 155)) + [-300, -250, 200, 300, 303], 40, 1)
    for (b, sigma, d), n in zip(cases, skip([(b, s, d * d) for b, s, d in cases])):
        assert 0 <= n < 20_000
        # the tip comes at most b closer per step, and b + sigma is near
        assert n == 0 or Fraction(b) * (n + 1) + Fraction(sigma) <= Fraction(d), (b, sigma, d, n)


def test_skips_what_it_can(skip):
    cases = _cases(range(-140, 140), 40, 2)
    for (b, sigma, d), n in zip(cases, skip([(b, s, d * d) for b, s, d in cases])):
        allowed = math.floor(d / b - 1.0 - sigma / b)
        assert n >= min(allowed * 0.999, 16_384) - 1.0 - 1e-6, (b, sigma, d, n)


def test_values_that_are_no_number_of_steps(skip):
    inf, nan = math.inf, math.nan
    cases = [(1.0, 1.0, inf), (1.0, 1.0, nan), (1e18, 1e18, inf), (1e-200, 1e-200, 1e-300), (1e-200, 0.0, 0.0),
             (1e200, 1e200, inf), (1e200, 0.0, 1e300), (1.0, 1e300, inf), (1e-300, 1e300, 1.0), (1.0, 1e200, 1e308)]
    assert skip(cases) == [0] * len(cases)
