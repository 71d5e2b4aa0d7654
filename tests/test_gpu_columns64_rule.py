"""Many right-hand sides of FP64 matrices at both sides of the rule for four
wavefronts per item: sweeps of 512 and 1,024 items with a short streaming
list, and sweeps of 128 and less.  FP64 sums of at most some 10^4 products per row
in another order than the single-vector product's: 1e-13."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [False, True], ids=["full", "half"])
@pytest.mark.parametrize("n,leaf,p,nrhs", [(9000, 9, 3, 16), (9000, 18, 4, 32), (4000, 33, 5, 19)])
def test_columns_match_single_products(n, leaf, p, nrhs, half):
    from paper_1902_01829_amd import h2mv
    print(f"case n={n} leaf={leaf} p={p} nrhs={nrhs} half={half}", flush=True)
    A = h2mv.H2Matrix(np.random.default_rng(n).random((n, 2)), 2, leaf, p, 0.9, 0.1,
                      storage=h2mv.H2_HALF_STORAGE if half else 0)
    X = torch.randn(nrhs, n, dtype=torch.float64, device="cuda")
    Y = A.matmat(X)
    assert torch.equal(Y, A.matmat(X))
    for j in (0, 1, nrhs - 1):
        y = A.matvec(X[j].contiguous())
        assert (Y[j] - y).norm().item() <= 1e-13 * y.norm().item(), j
    A.close()
