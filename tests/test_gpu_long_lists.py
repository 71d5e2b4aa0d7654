"""The block loops of the streaming launch with 32-wide tiles on ragged blocks.

Short lists, 16-wide tiles and FP32 batches stream by mm_stream_tiles_kernel
whatever the launch shape, so the loops behind the pinned depths 0 to 5 run
only in lists longer than the rule in h2_mm.hip names (8,192 pair items in FP32,
4,096 in BF16): matrices of 2,048 and 4,096 leaves, with the length checked
against that rule.  Rows and widths that are no multiple of 8, 16 or 32.

Tolerance: FP32 block products of at most 64 terms (2^-24 * 64 * |a||x| with
random signs, about 1e-7 of a row) under FP64 sums, against the oracle on the
same dequantized values: 1e-6.  The depths run a block's products and the sums
over blocks in one order: equal bits."""
import os
import re

import numpy as np
import pytest

from paper_1902_01829_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# leaves of 38-39 points, rank 49 (a row per workgroup); leaves of 21-22 points, rank 25 (two rows)
CASES = [W.C1.with_(name="2d-n78900-m41-p7", n=78900, leaf=41, cheb_p=7, seed=951),
         W.C1.with_(name="2d-n88500-m23-p5", n=88500, leaf=23, cheb_p=5, seed=952)]


def _rule():
    """The most pair items of a list that streams by tiles: {storage: items}."""
    with open(os.path.join(ROOT, "paper_1902_01829_amd", "csrc", "h2_mm.hip")) as f:
        body = re.search(r"static bool stream_by_tiles\(.*?\n\}", f.read(), re.S).group(0)
    fp32, bf16 = (int(v) for v in re.findall(r"npitems <= (\d+)", body))
    return {1: fp32, 2: bf16}


def _pair_items(A, w):
    """Pair items of the streaming list without its padding: two per row of more than 32 rows."""
    i = A.info
    m = -(-w.n >> i.levels_q)   # rows of the largest leaf
    nodes = (2 << i.levels_q) - (1 << i.lmin)
    return sum(rows * (2 if size > 32 else 1) for rows, size in ((nodes, i.rank), (1 << i.levels_q, m)))


@pytest.mark.parametrize("storage", [1, 2], ids=["fp32", "bf16"])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_every_depth_on_ragged_long_lists(oracle_mod, w, storage):
    from paper_1902_01829_amd import h2mv
    A = h2mv.H2Matrix(W.points(w), w.dim, w.leaf, w.cheb_p, w.eta, w.corr_len, storage=storage)
    assert _pair_items(A, w) > _rule()[storage], "the block loops no longer run here"
    print(f"case {w.name} storage {storage}: {_pair_items(A, w)} pair items", flush=True)
    o = oracle_mod.OracleH2(W.points(w), w.leaf, w.cheb_p, w.eta, w.corr_len, storage=storage, keep_blocks=False)
    for nrhs in (20, 32):
        X = np.random.default_rng(w.n + nrhs).standard_normal((nrhs, w.n))
        Xd = torch.from_numpy(X).cuda()
        first = None
        for depth in range(6):
            for grid in (0, 256):
                A.set_matmat_tuning(0, depth, 32, grid)
                Y = A.matmat(Xd)
                if first is None:
                    first = Y
                    for j in (0, nrhs - 1):
                        ref = o.matvec(X[j])
                        rel = np.linalg.norm(Y[j].cpu().numpy() - ref) / np.linalg.norm(ref)
                        print(f"  {nrhs} right-hand sides, column {j}: {rel:.2e}", flush=True)
                        assert rel <= 1e-6
                assert torch.equal(Y, first), (nrhs, depth, grid)
    A.close()


def test_every_depth_on_a_long_bf16_batch():
    """The same loops with a batch's addresses: each member's own product."""
    from paper_1902_01829_amd import h2mv
    mats = [h2mv.H2Matrix(W.points(w), w.dim, w.leaf, w.cheb_p, w.eta, w.corr_len, storage=2) for w in CASES]
    assert sum(_pair_items(A, w) for A, w in zip(mats, CASES)) > _rule()[2], "the block loops no longer run here"
    Xs = [torch.randn(20, A.n, dtype=torch.float64, device="cuda") for A in mats]
    batch, refs = h2mv.H2Batch(mats, 20), []
    for A, X in zip(mats, Xs):
        A.set_matmat_tuning(0, 0, 32, 0)
        refs.append(A.matmat(X))
    for depth in range(6):
        for grid in (0, 256):
            batch.set_tuning(depth, grid, 32)
            for Y, ref in zip(batch.matmat(Xs), refs):
                rel = ((Y - ref).norm() / ref.norm()).item()
                assert rel <= 1e-12, (depth, grid, rel)
    batch.close()
    for A in mats:
        A.close()
