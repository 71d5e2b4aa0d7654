"""Compression at the edges of the basis generation's and the truncation's
shapes: ranks around the 16-column slots of a wavefront (1 to 9, 25, 36, 49,
64), odd ranks, and stacks of one to several
passes (up to 448 appended rows each), against the oracle's compress_arrays.

Ranks are counts of singular values above a threshold and must be equal (no
singular value within a relative 1e-6 of it).  The products may differ by
rounding, 2^-53 times the rows of a stack (under 10^4) over the gap at a cut
(1e-4 or more in these cases): 1e-11, checked on both compressed matrices."""
import numpy as np
import pytest

from paper_1902_01829_amd import workloads as W
from test_gpu_compress import PARITY_TOL, _check_margin, _rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [(2, 1, 900, 16, 1e-3), (2, 3, 1500, 32, 1e-4), (2, 5, 2500, 64, 1e-5), (2, 6, 3000, 64, 1e-5),
         (2, 7, 3600, 64, 1e-6), (3, 1, 1200, 16, 1e-2), (3, 2, 2500, 24, 1e-3), (3, 4, 4096, 64, 1e-3)]


@pytest.mark.parametrize("dim,p,n,leaf,eps", CASES)
def test_compress_ranks_and_products(oracle_mod, dim, p, n, leaf, eps):
    from paper_1902_01829_amd import h2mv
    w = W.C1.with_(n=n, dim=dim, leaf=leaf, cheb_p=p, corr_len=0.1 * (dim - 1), seed=700 + 10 * p + dim)
    o = oracle_mod.OracleH2(W.points(w), w.leaf, w.cheb_p, w.eta, w.corr_len)
    ref, info = oracle_mod.compress_arrays(o.export_arrays(), eps)
    _check_margin(info, eps)
    A = h2mv.H2Matrix(W.points(w), w.dim, w.leaf, w.cheb_p, w.eta, w.corr_len, storage=0)
    ranks = A.compress(eps)
    x = W.rhs(w)[o.perm()]
    d = _rel(A.matvec(torch.from_numpy(x).cuda()).cpu().numpy(), oracle_mod.arrays_matvec(ref, x))
    print(f"ranks {[int(r) for r in ranks]}, product vs oracle {d:.2e}", flush=True)
    A.close()
    assert [int(r) for r in ranks] == [int(r) for r in ref["level_rank"]]
    assert d <= PARITY_TOL
