"""Many right-hand sides of FP64 matrices on the FP64 matrix cores: edges of
the tiles (rows of 1 to 64, odd widths, 16- and 32-wide passes), both ways
of spreading a list's items over wavefronts, and the two cases that keep
the single-vector products (no memory for the tiles, first call under capture)."""
import os

import numpy as np
import pytest

from paper_1902_01829_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# FP64 sums of at most some 10^4 products per row in another order than the
# single-vector product's: rounding grows like sqrt(10^4) 2^-53 = 1e-14.
TOL = 1e-13

CASES = [
    (1, 2, 4, 3, 2), (5, 2, 2, 3, 17), (65, 2, 64, 8, 16), (777, 2, 24, 3, 15), (3000, 3, 24, 3, 33),
    (5003, 2, 37, 7, 31), (4000, 3, 64, 4, 65),
    (70000, 2, 16, 3, 3),    # more items than the four-wavefront rule takes
    (300000, 2, 33, 5, 17),
]


def _build(n, dim, leaf, p, half=False):
    from paper_1902_01829_amd import h2mv
    pts = np.random.default_rng(n).random((n, dim))
    return h2mv.H2Matrix(pts, dim, leaf, p, 0.9, 0.1, storage=h2mv.H2_HALF_STORAGE if half else 0)


@pytest.mark.parametrize("half", [False, True], ids=["full", "half"])
@pytest.mark.parametrize("n,dim,leaf,p,nrhs", CASES)
def test_columns_match_single_products(n, dim, leaf, p, nrhs, half):
    print(f"case n={n} dim={dim} leaf={leaf} p={p} nrhs={nrhs} half={half}", flush=True)
    A = _build(n, dim, leaf, p, half)
    X = torch.randn(nrhs, n, dtype=torch.float64, device="cuda")
    Y = A.matmat(X)
    assert torch.equal(Y, A.matmat(X))   # the sums keep their order from call to call
    for j in sorted({0, 1, nrhs // 2, nrhs - 1}):
        y = A.matvec(X[j].contiguous())
        assert (Y[j] - y).norm().item() <= TOL * y.norm().item(), j
    A.close()


def test_infinities_stay_in_their_column():
    """An infinite input value reaches what it reaches in the single-vector
    product and no other right-hand side."""
    A = _build(777, 2, 24, 3)
    X = torch.randn(5, 777, dtype=torch.float64, device="cuda")
    ref = A.matmat(X)
    X[2, 100] = float("inf")
    Y = A.matmat(X)
    y = A.matvec(X[2].contiguous())
    assert torch.equal(torch.isfinite(Y[2]), torch.isfinite(y)) and torch.equal(torch.isnan(Y[2]), torch.isnan(y))
    for j in (0, 1, 3, 4):
        assert torch.equal(Y[j], ref[j])
    A.close()


def test_leading_dimensions_and_unaligned_columns():
    from paper_1902_01829_amd import h2mv
    n, r = 777, 6
    A = _build(n, 2, 24, 3)
    X = torch.randn(r * (n + 3) + 1, dtype=torch.float64, device="cuda")
    Y = torch.full((r * (n + 5) + 1,), 7.0, dtype=torch.float64, device="cuda")
    h2mv.h2_matmat(A.handle, X.data_ptr() + 8, n + 3, Y.data_ptr() + 8, n + 5, r,
                   torch.cuda.current_stream().cuda_stream)
    Xc = torch.stack([X[1 + j * (n + 3):1 + j * (n + 3) + n] for j in range(r)])
    ref = A.matmat(Xc.contiguous())
    for j in range(r):
        o = 1 + j * (n + 5)
        assert torch.equal(Y[o:o + n], ref[j])
        assert bool((Y[o + n:o + n + 5] == 7.0).all()) or j == r - 1
    assert Y[0].item() == 7.0
    A.close()


def test_no_memory_for_tiles_runs_single_products():
    from paper_1902_01829_amd import h2mv
    n = 4096
    A = _build(n, 2, 32, 4)
    total = A.info.bytes_device_total
    A.close()
    os.environ["H2MV_DEVICE_BYTE_CAP"] = str(total + 4096)
    try:
        A = _build(n, 2, 32, 4)
    finally:
        os.environ.pop("H2MV_DEVICE_BYTE_CAP")
    X = torch.randn(4, n, dtype=torch.float64, device="cuda")
    Y = A.matmat(X)
    for j in range(4):
        assert torch.equal(Y[j], A.matvec(X[j].contiguous()))
    assert A.info.bytes_device_total == total and h2mv.h2_get_info(A.handle).n == n
    A.close()


def test_first_call_under_capture():
    n = 4096
    A = _build(n, 2, 32, 4)
    X = torch.randn(4, n, dtype=torch.float64, device="cuda")
    Y = torch.empty_like(X)
    A.matvec(X[0].contiguous())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.matmat(X, out=Y)
    for k in range(3):
        X.copy_(torch.randn_like(X))
        Y.zero_()
        g.replay()
        torch.cuda.synchronize()
        ref = A.matmat(X)   # the tiles are there now: matrix cores
        assert ((Y - ref).norm() / ref.norm()).item() <= TOL
    g2 = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g2):
        A.matmat(X, out=Y)
    for k in range(3):
        X.copy_(torch.randn_like(X))
        g2.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, A.matmat(X))
    A.close()
