"""The rule that gives hard-sphere calls to the queued or to the lockstep kernel:
the call is not slower than on the lockstep kernel, which a tuning table entry
selects, and ensembles large enough for the queued kernel where small ones stay
with the other agree with the oracle bit for bit (Sec. 3.3.3).  GPU test; calls
the HIP library through its C ABI.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1704_04381_amd as rs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _clean_table():
    rs.mapping_clear()
    yield
    rs.mapping_clear()


def _ms(N, k, M, sigma):
    best = float("inf")
    rs.kernel_timing(True)
    for _ in range(8):
        rs.kernel_time()
        rs.gen_chains("real", N, k, M, 7, sync=False, bead_diameter=sigma)
        torch.cuda.synchronize()
        best = min(best, rs.kernel_time()[0])
    rs.kernel_timing(False)
    return best


@pytest.mark.parametrize("N,k,M,sigma", [
    (100, 4, 64_000, 0.6),     # long-lived chains of few trials
    (279, 1, 30_000, 1.0),     # chains that end at once, at the end of the lockstep
    (500, 2, 60_000, 1.0),     # loop's early exit and beyond
    (1_000, 1, 30_000, 1.0),
    (280, 8, 32_000, 0.4),     # 64 lanes, few dead ends
    (180, 8, 30_000, 0.75),
    (200, 6, 8_000, 0.9),
    (400, 8, 1_000, 1.0),
])
def test_rule_is_not_slower_than_lockstep(N, k, M, sigma):
    # 1.5 to 3 times slower before the rule looked at M and sigma, or at most
    # 1.1 times with it; the line lies between, well above the timing's noise
    print(f"[gpu] real rule N={N} k={k} M={M} sigma={sigma}", flush=True)
    rule = _ms(N, k, M, sigma)
    q = rs.mapping_query(rs.make_config("real", N, k, M, 7, bead_diameter=sigma))
    rs.mapping_set("real", k, N, N, q["lanes"], q["threads"])
    lockstep = _ms(N, k, M, sigma)
    print(f"rule {rule:.3f} ms, lockstep {lockstep:.3f} ms")
    assert rule < 1.15 * lockstep


def _ends_match(out, sp):
    M, n = sp["n_chains"], 12
    for first in (0, M // 2, M - n):
        ref = oracle.gen_real(sp["seed"], sp["N"], sp["k"], n, chain_offset=first)
        for key in ("log_w", "r2", "rg2"):
            np.testing.assert_array_equal(out[key].cpu().numpy()[first:first + n], ref[key], err_msg=key)
        np.testing.assert_array_equal(out["r_end"].cpu().numpy()[:, first:first + n], ref["r_end"])
        np.testing.assert_array_equal(out["n_grown"].cpu().numpy().view(np.uint16)[first:first + n], ref["n_grown"])


@pytest.mark.parametrize("N,k,M", [(144, 8, 130_000), (213, 8, 70_001), (279, 8, 70_000), (280, 8, 30_000),
                                   (400, 16, 6_003), (100, 4, 70_000)])
def test_large_ensembles_bit_exact(N, k, M):
    print(f"[gpu] real rule N={N} k={k} M={M}", flush=True)
    out, s = rs.gen_chains("real", N, k, M, 341)
    torch.cuda.synchronize()
    _ends_match(out, dict(N=N, k=k, n_chains=M, seed=341))
    assert s["n_alive"] == int(np.isfinite(out["log_w"].cpu().numpy()).sum())


def test_ensembles_of_a_batch_count_together():
    specs = [dict(geometry="real", N=N, k=8, n_chains=45_000, seed=350 + N) for N in (144, 213, 60, 300)]
    print("[gpu] real rule batch", flush=True)
    for sp, (out, _s) in zip(specs, rs.gen_batch(specs)):
        torch.cuda.synchronize()
        _ends_match(out, sp)
