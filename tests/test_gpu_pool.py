"""Device memory that outlives a handle: matrices made and dropped in turn (the
next ones get the memory of the last) give bitwise the products of the first,
on several host threads at once."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _build(n):
    from paper_1902_01829_amd import h2mv
    return h2mv.H2Matrix(np.random.default_rng(n).random((n, 2)), 2, 64, 5, 0.9, 0.1)


def test_reused_memory_gives_the_same_products():
    import gc
    gc.collect()
    torch.cuda.synchronize()
    keep = _build(3000)
    ns = (9000, 20000, 8000)
    x = {n: torch.from_numpy(np.random.default_rng(n + 1).standard_normal(n)).cuda() for n in ns}
    ref, bad = {}, []
    for n in ns:
        A = _build(n)
        ref[n] = A.matvec(x[n]).clone()
        A.close()

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(6):
                n = ns[(i + k) % len(ns)]
                A = _build(n)
                y = A.matvec(x[n])
                T = A.transpose()
                z = T.matvec(x[n])
                torch.cuda.current_stream().synchronize()
                if not torch.equal(y, ref[n]) or float((z - ref[n]).norm() / ref[n].norm()) > 1e-12:
                    bad.append((i, k, n))
                T.close()
                A.close()

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    keep.close()
