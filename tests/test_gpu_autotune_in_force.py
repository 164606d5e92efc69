"""rsaw_autotune where the kernel in force has no lane mapping: nothing that would
replace it is reported as chosen or installed unless it was faster.  GPU test;
calls the HIP library through its C ABI.
"""
import pytest

torch = pytest.importorskip("torch")

import paper_1704_04381_amd as rs

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _clean_table():
    rs.mapping_clear()
    yield
    rs.mapping_clear()


@pytest.mark.parametrize("geo,k,edge", [("lattice", 6, 6_000), ("lattice26", 26, 3_000)])
def test_site_set_stays_and_is_not_reported_as_a_mapping(geo, k, edge):
    # the site set is 5 to 10 times as fast as any mapping here
    print(f"[gpu] autotune in force {geo} N={edge}", flush=True)
    r, = rs.autotune(geo, k, [edge], 500, reps=1)
    assert r["k_trials"] == 0 and r["ms"] > 0.0
    assert rs.mapping_list() == []
    with pytest.raises(rs.RsawError):
        rs.mapping_set(geo, r["k_trials"], r["n_lo"], r["n_hi"], r["lanes"], r["threads"])


def test_winning_mapping_is_reported_with_its_k():
    print("[gpu] autotune in force lattice N=100", flush=True)
    r, = rs.autotune("lattice", 6, [100], 2_000, reps=1)
    assert r["k_trials"] == 6
