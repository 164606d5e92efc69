"""The site-set kernel of long lattice chains against the oracle, bit for bit
(Sec. 3.3.2), on the simple cubic and the 26-neighbour lattice: the edges of the rule that selects it, chains per wave from
eight to one, restarts, chain offsets past 2^32, ensembles smaller than a
wave, several ensembles in a launch, and, with the byte box lowered, chains
that are grown again without the set.  The calls repeat within a process, so
the chain queue starts each from zero.  GPU test; calls the HIP library
through its C ABI.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1704_04381_amd as rs
from test_gpu_parity import _lattice_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _restore():
    yield
    rs.set_byte_box(0)


@pytest.mark.parametrize("N,M,seed,coord,edge,offset,restart", [
    (2_049, 1, 201, "i32", 0, 0, False),
    (1_025, 700, 202, "i16", 0, 0, True),
    (2_100, 150, 203, "i32", 0, (1 << 32) + 11, False),
    (1_025, 4_096, 204, "i16", 0, 0, False),  # the rule's smallest ensemble
    (513, 1_500, 205, "i32", 0, 0, True),     # its shortest chains
    (5_000, 25, 206, "i16", 0, 0, False),
    (16_384, 5, 207, "i32", 0, 0, False),     # the longest
    (2_060, 90, 208, "i32", 40, 0, False),    # some chains without the set
    (1_030, 40, 209, "i16", 1, 7, True),      # all of them
])
def test_site_set_bit_exact(N, M, seed, coord, edge, offset, restart):
    rs.set_byte_box(edge)
    _lattice_case(N, M, seed, coord=coord, bins=64, offset=offset, restart=restart)


@pytest.mark.parametrize("N,M,seed,coord,edge,offset,restart", [
    (301, 500, 221, "i16", 0, 0, False),      # the rule's shortest chains
    (301, 9, 222, "i32", 0, (1 << 32) + 3, True),
    (700, 100, 223, "i32", 0, 0, False),
    (2_049, 12, 224, "i16", 0, 0, False),
    (9_000, 3, 225, "i32", 0, 0, False),
    (310, 150, 226, "i16", 25, 0, False),     # some chains without the set
    (400, 40, 227, "i32", 1, 5, True),        # all of them
])
def test_site_set26_bit_exact(N, M, seed, coord, edge, offset, restart):
    from test_gpu_lattice26 import _case
    rs.set_byte_box(edge)
    _case(N, M, seed, coord=coord, bins=64, offset=offset, restart=restart)


@pytest.mark.parametrize("geometry,N,M", [
    ("lattice", 1_100, 16_000),   # eight chains per wave, small tables
    ("lattice", 2_500, 7_000),    # five
    ("lattice", 8_000, 1_700),    # two, a wave per SIMD
    ("lattice26", 512, 21_000),
    ("lattice26", 1_900, 6_500),
    ("lattice26", 6_000, 2_300),
])
def test_site_set_ensembles_that_fill_the_lds(geometry, N, M):
    """The smallest tables, which calls of many chains take: their first and
    last chains against the oracle."""
    out, s = rs.gen_chains(geometry, N, 26 if geometry == "lattice26" else 6, M, 231)
    torch.cuda.synchronize()
    n = 12
    for first in (0, M - n):
        ref = oracle.gen_lattice(231, N, n, chain_offset=first, z26=geometry == "lattice26")
        for key in ("log_w", "n2rg2"):
            np.testing.assert_array_equal(out[key].cpu().numpy()[first:first + n], ref[key])
        np.testing.assert_array_equal(out["r_end"].cpu().numpy()[:, first:first + n].astype(np.int32), ref["r_end"])
        np.testing.assert_array_equal(out["n_grown"].cpu().numpy().view(np.uint16)[first:first + n], ref["n_grown"])
    assert s["n_alive"] == int(np.isfinite(out["log_w"].cpu().numpy()).sum())


def test_site_set_in_a_batch():
    specs = [dict(geometry="lattice", N=2_200, k=6, n_chains=60, seed=211),
             dict(geometry="lattice", N=3_000, k=6, n_chains=20, seed=212, coord="i16"),
             dict(geometry="lattice", N=1_026, k=6, n_chains=130, seed=213, restart=True),
             dict(geometry="lattice", N=300, k=6, n_chains=100, seed=214),
             dict(geometry="lattice26", N=330, k=26, n_chains=90, seed=215),
             dict(geometry="lattice26", N=900, k=26, n_chains=20, seed=216, coord="i16")]
    for _ in range(2):
        print("[gpu] site-set batch", flush=True)
        res = rs.gen_batch(specs)
        torch.cuda.synchronize()
        for sp, (out, s) in zip(specs, res):
            ref = oracle.gen_lattice(sp["seed"], sp["N"], sp["n_chains"], restart=sp.get("restart", False),
                                     z26=sp["geometry"] == "lattice26")
            np.testing.assert_array_equal(out["n_grown"].cpu().numpy().view(np.uint16), ref["n_grown"])
            np.testing.assert_array_equal(out["log_w"].cpu().numpy(), ref["log_w"])
            np.testing.assert_array_equal(out["r_end"].cpu().numpy().astype(np.int32), ref["r_end"])
            np.testing.assert_array_equal(out["n2rg2"].cpu().numpy(), ref["n2rg2"])
            assert s["n_alive"] == int(np.isfinite(ref["log_w"]).sum())
