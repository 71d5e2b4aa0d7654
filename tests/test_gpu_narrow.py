"""Many right-hand sides at the edges of the streaming launch's shapes (16-wide
tiles, and 32-wide ones in short lists): rows of 1 to 4 tiles of 16, block widths that are no multiple
of a chunk (16 columns, BF16 32), rows without blocks of a wavefront's share,
and rows whose share exceeds the 64 block descriptors loaded at a time (3-D,
small leaves), against the oracle on the same dequantized values.

Tolerance: a block's products add at most 64 terms in FP32 (2^-24 * 64 * |a||x|,
random signs: about 1e-7 of a row), the sums over blocks are FP64: 1e-6."""
import numpy as np
import pytest

from paper_1902_01829_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [(2, 1, 300, 3, 2), (2, 4, 900, 16, 16), (2, 4, 1000, 17, 1), (2, 5, 2000, 33, 8), (2, 7, 3000, 50, 9),
         (2, 8, 1500, 64, 16), (3, 3, 12000, 12, 3), (3, 2, 4000, 8, 5), (3, 4, 6000, 47, 15), (2, 3, 20, 64, 4),
         (2, 4, 900, 17, 17), (2, 7, 1500, 50, 32), (2, 8, 1000, 64, 20), (3, 2, 3000, 8, 31), (3, 3, 5000, 30, 40)]


@pytest.mark.parametrize("storage", [1, 2], ids=["fp32", "bf16"])
@pytest.mark.parametrize("dim,p,n,leaf,nrhs", CASES)
def test_narrow_passes(oracle_mod, dim, p, n, leaf, nrhs, storage):
    from paper_1902_01829_amd import h2mv
    w = W.C1.with_(n=n, dim=dim, leaf=leaf, cheb_p=p, corr_len=0.1 * (dim - 1), seed=800 + n)
    A = h2mv.H2Matrix(W.points(w), w.dim, w.leaf, w.cheb_p, w.eta, w.corr_len, storage=storage)
    X = np.random.default_rng(n + nrhs).standard_normal((nrhs, n))
    Y = A.matmat(torch.from_numpy(X).cuda()).cpu().numpy()
    A.close()
    o = oracle_mod.OracleH2(W.points(w), w.leaf, w.cheb_p, w.eta, w.corr_len, storage=storage, keep_blocks=True)
    worst = 0.0
    for j in sorted({0, nrhs // 2, nrhs - 1}):
        ref = o.matvec(X[j])
        worst = max(worst, float(np.linalg.norm(Y[j] - ref) / np.linalg.norm(ref)))
    print(f"worst column {worst:.2e}", flush=True)
    assert worst <= 1e-6
