"""The structure at the sizes where its construction goes over to several host
threads (8,192 points), with many equal coordinates and a deep tree:
identical to the oracle's."""
import numpy as np
import pytest

from paper_1902_01829_amd import h2mv


@pytest.mark.parametrize("n,dim,leaf,grid", [(8191, 2, 32, 0), (8192, 2, 33, 0), (8193, 3, 64, 0), (9000, 2, 2, 0),
                                             (20000, 3, 48, 12), (30011, 2, 24, 200)])
def test_structure_of_threads_identical_to_oracle(oracle_mod, n, dim, leaf, grid):
    pts = np.random.default_rng(n + dim).random((n, dim))
    if grid:
        pts = np.floor(pts * grid) / grid   # many points on each other
    o = oracle_mod.OracleH2(pts, leaf, 2, 0.9, 0.1, keep_blocks=False)
    h = h2mv.h2_build_from_points(pts, dim, leaf, 2, 0.9, 0.1, flags=h2mv.H2_FLAG_STRUCTURE_ONLY)
    try:
        assert np.array_equal(h2mv.h2_get_perm(h, n), o.perm())
        for l in range(o.q + 1):
            rp, ci = h2mv.h2_get_level_bsr(h, l, 1 << l)
            rp2, ci2 = o.coupling_bsr(l)
            assert np.array_equal(rp, rp2) and np.array_equal(ci, ci2), l
        rp, ci = h2mv.h2_get_level_bsr(h, -1, 1 << o.q)
        rp2, ci2 = o.dense_bsr()
        assert np.array_equal(rp, rp2) and np.array_equal(ci, ci2)
        assert h2mv.h2_get_info(h).near_ties == o.near_ties()
    finally:
        h2mv.h2_free(h)
