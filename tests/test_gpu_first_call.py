"""The first product of several columns on an FP64 handle, which makes its tile
workspace, while another stream of the process is being captured."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _build(n):
    from paper_1902_01829_amd import h2mv
    return h2mv.H2Matrix(np.random.default_rng(n).random((n, 2)), 2, 32, 4, 0.9, 0.1)


def test_first_columns_beside_another_streams_capture():
    """The capture goes on (torch's default: global mode), and the product is
    the one of a handle that made its workspace before."""
    n = 4096
    A, B = _build(n), _build(n)
    X = torch.randn(4, n, dtype=torch.float64, device="cuda")
    Y, ref = torch.empty_like(X), A.matmat(X)
    a = torch.ones(1000, device="cuda")
    side, run, g = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=side):
        a.mul_(2.0)
        with torch.cuda.stream(run):
            B.matmat(X, out=Y)
        a.add_(1.0)
    torch.cuda.synchronize()
    assert torch.equal(Y, ref) and bool((a == 1.0).all())
    for k in range(3):
        g.replay()
        B.matmat(X, out=Y)
    torch.cuda.synchronize()
    assert bool((a == 15.0).all()) and torch.equal(Y, ref)
    A.close()
    B.close()
