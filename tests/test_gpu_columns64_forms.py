"""Many right-hand sides of FP64 matrices of every form a handle can take:
compressed and orthogonalized (a rank per level), given by arrays with separate
row and column trees, transposed, without low-rank blocks, under the streamed
schedule, and compressed after the tiles were made.  FP64 sums of at most some
10^4 products per row in another order than the single-vector product's: 1e-13."""
import numpy as np
import pytest

from perf import cases

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _points(n, dim, leaf, p):
    from paper_1902_01829_amd import h2mv
    return h2mv.H2Matrix(np.random.default_rng(n).random((n, dim)), dim, leaf, p, 0.9, 0.1 * (dim - 1))


def _arrays(n, leaf, rank):
    from paper_1902_01829_amd import h2mv
    return h2mv.H2Matrix.from_arrays(cases._curve_arrays(dict(n=n, leaf=leaf, rank=rank), n), h2mv.H2_FP64)


def _compressed(A, eps):
    A.matmat(torch.randn(3, A.n, dtype=torch.float64, device="cuda"))   # tiles of the ranks before
    A.compress(eps)
    return A


def _orthogonal(A):
    A.matmat(torch.randn(3, A.n, dtype=torch.float64, device="cuda"))
    A.orthogonalize()
    return A


def _streamed(A):
    from paper_1902_01829_amd import h2mv
    A.set_schedule(h2mv.H2_SCHEDULE_STREAMED)
    return A


FORMS = {
    "compressed-2d": lambda: _compressed(_points(6000, 2, 64, 6), 1e-5),
    "compressed-3d": lambda: _compressed(_points(5000, 3, 64, 3), 1e-3),
    "orthogonalized": lambda: _orthogonal(_points(5000, 2, 48, 5)),
    "arrays": lambda: _arrays(5003, 37, 9),
    "arrays-transposed": lambda: _arrays(5003, 37, 9).transpose(),
    "points-transposed": lambda: _points(3001, 2, 29, 4).transpose(),
    "one-leaf": lambda: _points(50, 2, 64, 3),
    "streamed": lambda: _streamed(_points(5000, 2, 33, 5)),
}


@pytest.mark.parametrize("form", list(FORMS))
def test_columns_match_single_products(form):
    print(f"form {form}", flush=True)
    A = FORMS[form]()
    for nrhs in (2, 16, 19, 33):
        X = torch.randn(nrhs, A.n, dtype=torch.float64, device="cuda")
        Y = A.matmat(X)
        for j in sorted({0, nrhs // 2, nrhs - 1}):
            y = A.matvec(X[j].contiguous())
            assert (Y[j] - y).norm().item() <= 1e-13 * y.norm().item(), (nrhs, j)
    A.close()
