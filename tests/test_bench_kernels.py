"""The growth kernel that bench.py prices a workload at is the one that the
library's rules choose; host-only calls of the HIP library."""
import os
import sys

import pytest

import paper_1704_04381_amd as rs

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def _model(geometry, N, k, n_chains, **kw):
    if not os.path.exists(rs.LIB_PATH):
        pytest.skip("librsaw.so not built")
    rs.mapping_clear()
    coord = "f64" if geometry == "real" else "i32"
    return bench.path_model(dict(geometry=geometry, N=N, k=k, n_chains=n_chains, seed=1, coord=coord, **kw))


@pytest.mark.parametrize("geo,N,k,M,kw,kernel", [
    ("lattice", 64, 6, 1_000, {}, "grow_lattice_reg"),
    ("lattice", 28, 6, 1_000, dict(exact_w=True), "grow_lattice_reg"),
    ("lattice", 600, 6, 1_000, {}, "grow_lattice_grp"),
    ("lattice", 600, 6, 1_000, dict(restart=True), "grow_lattice_set"),
    ("lattice", 2_000, 6, 4_000, {}, "grow_lattice_grp"),
    ("lattice", 2_000, 6, 5_000, {}, "grow_lattice_set"),
    ("lattice26", 64, 26, 1_000, {}, "grow_lattice26_lane"),
    ("lattice26", 300, 26, 1_000, {}, "grow_lattice26_grp"),
    ("lattice26", 301, 26, 1_000, {}, "grow_lattice_set"),
    ("real", 64, 8, 1_000_000, {}, "grow_real_tp"),
    ("real", 256, 8, 200_000, {}, "grow_real_queue"),
    ("real", 256, 8, 200_000, dict(bead_diameter=0.3), "grow_real_tp"),
    ("real", 3_000, 8, 3_000, {}, "grow_real_hbm"),
])
def test_kernel(geo, N, k, M, kw, kernel):
    assert _model(geo, N, k, M, **kw)["kernel"] == kernel


def test_register_kernels_are_priced_at_their_own_pair_test():
    assert bench.lattice_ops_per_chain(64) == 2 * 992 + 18 * 63 == 3118
    assert _model("lattice", 64, 6, 10)["ops"] == 31_180
