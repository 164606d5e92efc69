"""rsaw_set_byte_box and the site set: beyond N = 4096, where no kernel keeps one
word per monomer, and at edges that some format keeps anyway, it changes neither
results nor the time of a call.  GPU test; calls the HIP
library through its C ABI.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1704_04381_amd as rs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _restore():
    yield
    rs.set_byte_box(0)


def _run(geo, k, N, M):
    best = float("inf")
    rs.kernel_timing(True)
    for _ in range(3):
        rs.kernel_time()
        out, _s = rs.gen_chains(geo, N, k, M, 371)
        torch.cuda.synchronize()
        best = min(best, rs.kernel_time()[0])
    rs.kernel_timing(False)
    return best, {n: t.cpu().numpy() for n, t in out.items()}


@pytest.mark.parametrize("geo,k,N,M,edge", [
    ("lattice", 6, 5_000, 9, 60), ("lattice26", 26, 4_500, 5, 60),
    ("lattice", 6, 3_000, 60, 127), ("lattice26", 26, 2_048, 60, 62),
])
def test_no_effect_on_the_site_set(geo, k, N, M, edge):
    print(f"[gpu] byte box {geo} N={N} edge={edge}", flush=True)
    free, ref = _run(geo, k, N, M)
    rs.set_byte_box(edge)
    boxed, out = _run(geo, k, N, M)
    for name in ref:
        np.testing.assert_array_equal(out[name], ref[name], err_msg=name)
    # regrown chains would take N / 16 lookups' time per step instead of one's
    print(f"free {free:.3f} ms, boxed {boxed:.3f} ms")
    assert boxed < 3.0 * free
