"""The queued hard-sphere kernel against the oracle, every per-chain output bit
for bit (Sec. 3.3.3): each number of lanes at the edges of the rule that
selects it, trial counts off the powers of two, restarts, offsets past 2^32,
skipped blocks with other bond lengths and diameters, chains in global memory
around the LDS ring, and several ensembles in a launch.  GPU test; calls the
HIP library through its C ABI.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1704_04381_amd as rs

pytestmark = pytest.mark.gpu

KEYS = ("n_grown", "log_w", "r2", "rg2", "r_end")


def _same(out, ref, what):
    for key in KEYS:
        x = out[key].cpu().numpy()
        if key == "n_grown":
            x = x.view(np.uint16)
        np.testing.assert_array_equal(x, ref[key], err_msg=f"{what} {key}")


@pytest.mark.parametrize("N,k,M,seed,offset,restart,b,sigma", [
    (80, 4, 700, 301, 0, False, 1.0, 1.0),           # 16 lanes, 4 sets of trials
    (139, 1, 300, 302, 0, False, 1.0, 0.4),          # eight sets
    (140, 3, 300, 303, 3, False, 1.0, 0.75),         # 32 lanes, trials off a power of two
    (144, 8, 400, 304, (1 << 32) + 5, False, 1.0, 1.0),
    (150, 6, 60, 305, 0, True, 1.0, 0.6),            # restarts
    (279, 8, 130, 306, 0, False, 1.0, 1.0),
    (280, 8, 1, 307, 0, False, 1.0, 1.0),            # 64 lanes
    (400, 16, 60, 308, 0, False, 0.5, 0.45),
    (420, 4, 50, 309, 0, False, 2.5, 0.0),           # nothing overlaps: whole chains
    (500, 32, 25, 310, 0, False, 1.0, 1.0),
    (1_000, 64, 5, 311, 0, False, 1.0, 1.0),
    (1_536, 8, 40, 312, 0, False, 1.0, 0.8),         # the longest in LDS
    (1_537, 8, 40, 313, 0, False, 1.0, 0.8),         # global memory
    (2_500, 4, 12, 314, 0, False, 3.0, 1.0),
    (4_500, 16, 4, 315, 0, False, 1.0, 0.5),         # a second register of due steps
])
def test_queued_chains_bit_exact(N, k, M, seed, offset, restart, b, sigma):
    print(f"[gpu] real queue N={N} k={k} M={M}", flush=True)
    out, s = rs.gen_chains("real", N, k, M, seed, chain_offset=offset, restart=restart, bond_length=b,
                           bead_diameter=sigma)
    torch.cuda.synchronize()
    ref = oracle.gen_real(seed, N, k, M, b=b, sigma=sigma, chain_offset=offset, restart=restart)
    _same(out, ref, f"N={N} k={k}")
    assert s["n_alive"] == int(np.isfinite(ref["log_w"]).sum()) and s["status"] == 0


def test_queued_chains_in_a_batch():
    specs = [dict(geometry="real", N=N, k=k, n_chains=M, seed=320 + N)
             for N, k, M in ((100, 4, 150), (150, 8, 90), (260, 8, 40), (300, 8, 30), (60, 8, 100), (1_600, 8, 12),
                             (450, 16, 10))]
    for _ in range(2):
        print("[gpu] real queue batch", flush=True)
        res = rs.gen_batch(specs)
        torch.cuda.synchronize()
        for sp, (out, _s) in zip(specs, res):
            _same(out, oracle.gen_real(sp["seed"], sp["N"], sp["k"], sp["n_chains"]), sp["N"])
