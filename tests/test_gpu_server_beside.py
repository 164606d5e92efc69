"""A small request that arrives while a long one runs on the server's other
stream is served beside it, not after it, and both results are those of
stand-alone calls.  The long requests run in the kernels whose blocks stay
until their chains run out.  GPU test; calls the HIP library through its C ABI.
"""
import time

import pytest

torch = pytest.importorskip("torch")

import paper_1704_04381_amd as rs

pytestmark = pytest.mark.gpu

SMALL = [("lattice", 64, 6, 10_000), ("lattice", 256, 6, 10_000), ("real", 64, 8, 10_000)]


def _alone(geometry, N, k, M, seed):
    return rs.gen_chains(geometry, N, k, M, seed, per_chain=False)[1]


@pytest.mark.parametrize("long", [
    ("real", 256, 8, 1_500_000),      # 32 lanes per chain, about 0.1 s
    ("real", 160, 4, 4_000_000),      # 16 waves per CU
    ("lattice", 2048, 6, 800_000),    # site set
    ("lattice26", 400, 26, 4_000_000),
])
def test_small_requests_do_not_wait_for_a_long_one(long):
    print(f"[gpu] server beside {long}", flush=True)
    want = [_alone(*sp, 5) for sp in SMALL]
    with rs.Server(streams=2) as srv:
        for sp in SMALL:  # first use of the kernels
            srv.wait(srv.submit(*sp, 4))
        big = srv.submit(*long, 3)
        time.sleep(0.005)
        got = []
        for sp in SMALL:
            got.append(srv.wait(srv.submit(*sp, 5)))
            print(f"{sp}: {got[-1]['latency_us'] / 1e3:.2f} ms", flush=True)
        early = srv.poll(big) is None
        res = None if not early else srv.wait(big)
    assert early, "the long request ended before the small ones"
    for w, g in zip(want, got):
        for key in ("n_alive", "sum_w", "sum_w_r2", "r2_mean", "rg2_mean"):
            assert g[key] == w[key], key
    ref = _alone(*long, 3)
    for key in ("n_alive", "sum_w", "sum_w_r2", "r2_mean", "rg2_mean"):
        assert res[key] == ref[key], key
