"""Hard-sphere chains of extreme bond lengths against the oracle, every
per-chain output bit for bit (Sec. 3.3.3): the kernels that skip whole blocks
of beads while the tip is too far from them must do so for every bond length
a call may have, also where squared distances leave the range of binary32 or
of binary64.  GPU test; calls the HIP library through its C ABI.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import paper_1704_04381_amd as rs
from test_gpu_real_queue import _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [5e18, 1e18, 1e17, 1e-21, 5e-23, 1e-23, 1e-40, 1e60, 1e150, 1e-150, 1e-158])
@pytest.mark.parametrize("N,k,M,sigma", [
    (400, 8, 60, 1.0),     # beads in LDS
    (1_600, 8, 40, 0.85),  # in global memory
])
def test_extreme_bond_lengths_bit_exact(N, k, M, sigma, b):
    print(f"[gpu] real scale N={N} k={k} M={M} b={b}", flush=True)
    out, _ = rs.gen_chains("real", N, k, M, 331, bond_length=b, bead_diameter=sigma * b)
    torch.cuda.synchronize()
    ref = oracle.gen_real(331, N, k, M, b=b, sigma=sigma * b)
    _same(out, ref, f"N={N} b={b}")
