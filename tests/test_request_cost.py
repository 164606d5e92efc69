"""The cost model of the serving loop's size classes (request_cost.hpp), compiled
for the host, against growth-kernel times measured on one MI355X: within a factor
of two for every kernel that the built-in rules choose.
"""
import math
import os
import subprocess

import pytest

import paper_1704_04381_amd as rs

HERE = os.path.dirname(os.path.abspath(__file__))
REPO = os.path.dirname(HERE)

MEASURED = [  # geometry, N, k, chains, sigma / b, ms
    ("lattice", 64, 6, 10_000_000, 1, 1.131), ("lattice", 128, 6, 1_000_000, 1, 0.625),
    ("lattice", 256, 6, 1_000_000, 1, 2.146), ("lattice", 512, 6, 300_000, 1, 2.409),
    ("lattice", 1_000, 6, 200_000, 1, 6.169), ("lattice", 1_100, 6, 200_000, 1, 6.985),
    ("lattice", 2_048, 6, 100_000, 1, 9.549), ("lattice", 5_000, 6, 20_000, 1, 7.735),
    ("lattice", 10_000, 6, 5_000, 1, 6.675), ("lattice", 16_384, 6, 4_000, 1, 9.301),
    ("lattice26", 64, 26, 1_000_000, 1, 0.474), ("lattice26", 128, 26, 1_000_000, 1, 1.965),
    ("lattice26", 256, 26, 500_000, 1, 3.920), ("lattice26", 400, 26, 200_000, 1, 3.850),
    ("lattice26", 1_000, 26, 100_000, 1, 7.036), ("lattice26", 2_048, 26, 30_000, 1, 7.538),
    ("lattice26", 8_000, 26, 4_000, 1, 14.842),
    ("real", 16, 8, 1_000_000, 1, 1.391), ("real", 64, 8, 1_000_000, 1, 7.000), ("real", 64, 16, 500_000, 1, 5.225),
    ("real", 128, 8, 200_000, 1, 5.107), ("real", 256, 8, 200_000, 1, 13.450), ("real", 256, 4, 200_000, 1, 3.252),
    ("real", 500, 8, 100_000, 1, 13.112), ("real", 1_000, 8, 50_000, 1, 13.060),
    ("real", 3_000, 8, 20_000, 1, 7.020), ("real", 3_000, 4, 100_000, 1, 3.995),
    ("real", 1_000, 16, 50_000, 1, 35.097), ("real", 256, 8, 100_000, 0.3, 9.464),
    ("real", 1_000, 8, 20_000, 0.3, 20.320), ("real", 3_000, 8, 4_000, 0.3, 16.096),
]


@pytest.fixture(scope="module")
def estimate(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("cost") / "request_cost")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(REPO, "include"),
                           "-I", os.path.join(REPO, "paper_1704_04381_amd", "csrc"), "-o", exe,
                           os.path.join(HERE, "pins", "request_cost.cpp")])

    def run(cases):
        text = "\n".join(f"{rs.GEOMETRIES[g]} {N} {k} {M} {b} {s}" for g, N, k, M, b, s in cases)
        return [float(v) for v in subprocess.check_output([exe], input=text, text=True).split()]
    return run


def test_within_a_factor_of_two(estimate):
    got = estimate([(g, N, k, M, 1.0, s) for g, N, k, M, s, _ in MEASURED])
    for row, ms in zip(MEASURED, got):
        assert 0.5 < ms / row[-1] < 2.0, (row, ms)


def test_scale_and_limits(estimate):
    a, b, c, d = estimate([("real", 500, 8, 1_000, 1.0, 1.0), ("real", 500, 8, 1_000, 1e18, 1e18),
                           ("real", 500, 8, 1_000, 1.0, 0.0), ("real", 500, 8, 0, 1.0, 1.0)])
    assert a == pytest.approx(b) and math.isfinite(c) and c >= a and d == 0.0
