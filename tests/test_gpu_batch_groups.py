"""Which ensembles of a batch share a launch: one that fills the GPU by itself
keeps the LDS of its own chains, whichever kernel serves it, and small ones go
together.  The number of growth launches tells.  GPU test; calls the HIP library
through its C ABI.
"""
import pytest

torch = pytest.importorskip("torch")

import paper_1704_04381_amd as rs

pytestmark = pytest.mark.gpu


def _launches(specs):
    print(f"[gpu] batch groups {specs}", flush=True)
    rs.gen_batch(specs, per_chain=False)
    torch.cuda.synchronize()
    rs.kernel_timing(True)
    rs.kernel_time()
    rs.gen_batch(specs, per_chain=False)
    torch.cuda.synchronize()
    n = rs.kernel_time()[1]
    rs.kernel_timing(False)
    return n


def _real(N, k, M):
    return dict(geometry="real", N=N, k=k, n_chains=M, seed=N)


def _z26(N, M):
    return dict(geometry="lattice26", N=N, k=26, n_chains=M, seed=N)


@pytest.mark.parametrize("large,small", [
    (_real(300, 8, 40_000), _real(1_536, 8, 200)),   # 64 lanes: 7 KB of LDS beside 36 KB
    (_real(150, 8, 300_000), _real(270, 8, 300)),    # 32 lanes
    (_real(90, 4, 300_000), _real(139, 4, 300)),     # 16 lanes
    (_z26(301, 200_000), _z26(3_000, 100)),          # site sets
])
def test_a_large_queued_ensemble_is_launched_on_its_own(large, small):
    assert _launches([large]) == 1
    assert _launches([large, small]) == 2


def test_small_queued_ensembles_share_a_launch():
    assert _launches([_real(300, 8, 500), _real(1_200, 8, 200), _real(400, 8, 300)]) == 1
    assert _launches([_z26(301, 20_000), _z26(3_000, 100)]) == 1
