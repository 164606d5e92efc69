"""rsaw_mapping_query tells a mapping that a call runs with from one that a table
entry would only replace (k_trials 0), at the edges of the rules that give calls
to kernels without a mapping.  Host-only calls of the HIP library.
"""
import os

import pytest

import paper_1704_04381_amd as rs


@pytest.fixture(autouse=True)
def _clean_table():
    if not os.path.exists(rs.LIB_PATH):
        pytest.skip("librsaw.so not built")
    rs.mapping_clear()
    yield
    rs.mapping_clear()


@pytest.mark.parametrize("geo,N,k,M,kw,runs", [
    ("lattice", 2_048, 6, 1_000, {}, True),
    ("lattice", 2_049, 6, 1_000, {}, False),
    ("lattice", 1_025, 6, 4_095, {}, True),
    ("lattice", 1_025, 6, 4_096, {}, False),
    ("lattice", 512, 6, 1_000, dict(restart=True), True),
    ("lattice", 513, 6, 1_000, dict(restart=True), False),
    ("lattice26", 300, 26, 1_000, {}, True),
    ("lattice26", 301, 26, 1_000, {}, False),
    ("real", 143, 8, 200_000, {}, True),
    ("real", 144, 8, 200_000, {}, False),
    ("real", 144, 8, 200_000, dict(bead_diameter=0.4), True),
    ("real", 1_536, 8, 100, {}, False),
    ("real", 1_537, 8, 100, {}, True),
])
def test_query_says_whether_the_mapping_runs(geo, N, k, M, kw, runs):
    m = rs.mapping_query(rs.make_config(geo, N, k, M, 1, **kw))
    assert m["k_trials"] == (k if runs else 0)
    if not runs:
        # installed with a k of its own, the mapping replaces that kernel ...
        with pytest.raises(rs.RsawError):
            rs.mapping_set(geo, m["k_trials"], N, N, m["lanes"], m["threads"])
        rs.mapping_set(geo, k, N, N, m["lanes"], m["threads"])
        q = rs.mapping_query(rs.make_config(geo, N, k, M, 1, **kw))
        assert (q["k_trials"], q["lanes"], q["threads"]) == (k, m["lanes"], m["threads"])
