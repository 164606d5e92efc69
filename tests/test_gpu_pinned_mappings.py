"""The scanning group kernels at lengths where the built-in rules serve calls
with another kernel, pinned by a table entry: every per-chain output against the
oracle, bit for bit, with the words' own boxes and with lowered ones.  The
entries are the mappings of the kernels that the cases name, and the query says
that the call runs with them.  GPU test; calls the HIP library through its C ABI.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1704_04381_amd as rs
from test_gpu_lattice26 import _case as _lattice26_case
from test_gpu_parity import _lattice_case, _real_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _restore():
    rs.mapping_clear()
    yield
    rs.set_byte_box(0)
    rs.mapping_clear()


def _pin(geo, N, k, M, seed, lanes, **kw):
    """The built-in mapping of the scanning kernel, made the one in force."""
    cfg = rs.make_config(geo, N, k, M, seed, **kw)
    q = rs.mapping_query(cfg)
    assert q["lanes"] == lanes
    rs.mapping_set(geo, k, N, N, q["lanes"], q["threads"])
    now = rs.mapping_query(cfg)
    assert (now["k_trials"], now["lanes"], now["threads"]) == (k, q["lanes"], q["threads"])


@pytest.mark.parametrize("N,M,seed,coord,edge,lanes,offset,restart", [
    # byte words in registers, 16 to 64 lanes per chain
    (600, 60, 401, "i16", 0, 16, 0, True),
    (1_500, 40, 88, "i16", 35, 32, 0, True),
    (2_048, 60, 402, "i32", 0, 32, (1 << 32) + 9, False),
    (2_049, 40, 29, "i16", 0, 64, 0, False),
    (3_000, 12, 110, "i32", 60, 64, 0, False),
    (3_001, 16, 34, "i32", 0, 64, 0, False),
    # at the words' own edge: chain 5 of seed 1 reaches x = -134
    (4_096, 8, 1, "i16", 127, 64, 0, False),
    (4_096, 8, 1, "i32", 0, 64, 0, False),
    # just below it, where the tip is looked at every eight steps
    (4_096, 8, 1, "i16", 119, 64, 0, False),
    (2_049, 40, 34, "i16", 0, 64, 0, True),
    # two-word format in LDS
    (4_097, 8, 36, "i32", 0, 64, 0, False),
    (5_000, 12, 30, "i32", 0, 64, 0, False),
    (16_384, 2, 31, "i16", 0, 64, 0, False),
])
def test_six_neighbour_scan(N, M, seed, coord, edge, lanes, offset, restart):
    _pin("lattice", N, 6, M, seed, lanes, restart=restart)
    rs.set_byte_box(edge)
    out, _ = _lattice_case(N, M, seed, coord=coord, bins=64, offset=offset, restart=restart)
    # a lowered edge was reached by some chains, their ends show
    assert edge in (0, 119, 127) or (np.abs(out["r_end"].astype(np.int64)).max(axis=0) >= edge).sum() > 0


@pytest.mark.parametrize("N,M,seed,coord,edge,lanes,offset,restart", [
    # byte words to N = 640, packed words beyond, 8 to 64 lanes in registers
    (384, 200, 94, "i32", 30, 8, 0, False),
    (512, 150, 17, "i32", 0, 8, 0, False),
    (640, 60, 95, "i16", 40, 16, 0, False),
    (641, 50, 411, "i16", 0, 16, 0, False),
    (700, 80, 102, "i16", 30, 16, 0, False),
    (900, 24, 107, "i16", 0, 16, 0, False),
    (1_000, 40, 103, "i32", 40, 16, 0, True),
    (1_000, 65, 21, "i16", 0, 16, 0, False),
    (1_500, 30, 412, "i32", 45, 32, 0, False),
    (2_048, 16, 104, "i16", 60, 32, (1 << 32) + 5, False),
    (2_048, 12, 413, "i32", 0, 32, 0, False),
    (4_096, 4, 105, "i32", 100, 64, 0, False),
    (4_096, 4, 22, "i32", 0, 64, 0, False),
    # two-word format in LDS
    (4_097, 4, 23, "i16", 0, 64, 0, False),
    (16_384, 1, 25, "i16", 0, 64, 0, False),
])
def test_26_neighbour_scan(N, M, seed, coord, edge, lanes, offset, restart):
    _pin("lattice26", N, 26, M, seed, lanes, restart=restart)
    rs.set_byte_box(edge)
    out, _ = _lattice26_case(N, M, seed, coord=coord, bins=64, offset=offset, restart=restart)
    assert not edge or (np.abs(out["r_end"].astype(np.int64)).max(axis=0) >= min(edge, 62)).sum() > 0 or offset


@pytest.mark.parametrize("N,k,M,seed,lanes,sigma,restart", [
    (100, 4, 300, 421, 8, 1.0, False),
    (150, 8, 300, 51, 32, 1.0, False),
    (213, 8, 200, 52, 32, 1.0, False),
    (300, 8, 30, 33, 32, 1.0, True),
    (300, 5, 90, 16, 32, 1.0, False),
    (480, 3, 40, 18, 64, 1.0, False),
    (512, 16, 20, 50, 64, 0.8, False),
    (700, 8, 24, 42, 64, 1.0, False),
    (1_536, 8, 6, 51, 64, 0.5, False),
])
def test_hard_sphere_lockstep(N, k, M, seed, lanes, sigma, restart):
    _pin("real", N, k, M, seed, lanes, restart=restart, bead_diameter=sigma)
    _, s, exact = _real_case(N, k, M, seed, sigma=sigma, bins=64, restart=restart)
    assert exact and (not restart or s["n_alive"] == M)
