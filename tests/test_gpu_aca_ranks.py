"""The ACA kernels at ranks above the threads of a workgroup and above one load
of coefficients (128 and 64 terms), in single precision, and on blocks of more
rows than the 256-thread class takes, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import say


def _bin(lb, lo, hi):
    mx = np.maximum(lb[:, 1] - lb[:, 0], lb[:, 3] - lb[:, 2])
    pool = np.flatnonzero((mx > lo) & (mx <= hi))
    assert pool.size > 0, (lo, hi)
    return pool


@pytest.mark.parametrize("operator,precision,tol", [("collocation", "f64", 1e-12),
                                                    ("galerkin", "f64", 1e-12),
                                                    ("collocation", "f32", 2e-5)])
def test_ranks_above_the_workgroup(operator, precision, tol):
    """Fixed-rank mode (eps = 0) with max_rank 256 at N = 5,120 (leaf 64, eta 2):
    a block takes min(256, m, n) terms unless a residual is exactly zero before, the
    blocks of 320 rows twice as many as their workgroup has threads.  Entries agree
    to the rounding of the nodes (1e-13, in single precision 2e-6) and every further
    term leaves a residual of rounding size, so the factors reproduce the exact block
    to ten times that."""
    import paper_1806_11558_amd as hm
    from oracle import bem, galerkin
    from synthetic import icosphere
    V, T = icosphere(4)
    op = (bem.Operator if operator == "collocation" else galerkin.GalerkinOperator)(V, T)
    say("aca ranks", operator, precision)
    H = hm.HMatrix(V, T, leaf_size=64, eta=2.0, eps=0.0, max_rank=256, precision=precision,
                   operator=operator)
    lb, perm = H.lr_blocks(), H.perm()
    full = np.minimum(256, np.minimum(lb[:, 1] - lb[:, 0], lb[:, 3] - lb[:, 2]))
    assert np.all(lb[:, 4] <= full)
    assert np.all(lb[_bin(lb, 256, 512), 4] > 128)
    rng = np.random.default_rng(3)
    for lo, hi in ((0, 64), (64, 128), (128, 256), (256, 512)):
        for b in rng.choice(_bin(lb, lo, hi), 2, replace=False):
            r0, r1, c0, c1, rank, _ = lb[b]
            A = op.block(perm[r0:r1], perm[c0:c1])
            U, W = H.lr_factors(int(b))
            err = np.linalg.norm(A - U @ W.T) / np.linalg.norm(A)
            say("aca ranks", operator, precision, A.shape, int(rank), err)
            assert err <= tol
    H.free()


@pytest.mark.parametrize("precision,eps", [("f64", 1e-6), ("f32", 1e-3), ("f32", 1e-6)])
def test_largest_blocks_and_single_precision(precision, eps):
    """N = 81,920 (leaf 64, eta 2): one block of every size bin up to 4,096 rows and
    of those above (the 1,024-thread class), the rank of the oracle's ACA on exact
    rows and columns within one, 64 rows of the factors within 10 eps of exact
    ones.  (Single precision at eps = 1e-6 may go on for a few terms: its entries are
    rounded at 1e-7, and terms of that size are near the stop.)"""
    import paper_1806_11558_amd as hm
    from oracle import aca, bem
    from synthetic import icosphere
    V, T = icosphere(6)
    op = bem.Operator(V, T)
    say("aca bins", precision, eps)
    H = hm.HMatrix(V, T, leaf_size=64, eta=2.0, eps=eps, precision=precision)
    lb, perm = H.lr_blocks(), H.perm()
    rng = np.random.default_rng(5)
    for lo, hi in ((0, 64), (64, 128), (128, 256), (256, 512), (512, 1024), (1024, 2048),
                   (2048, 4096), (4096, 1 << 30)):
        b = int(rng.choice(_bin(lb, lo, hi)))
        r0, r1, c0, c1, rank, _ = lb[b]
        rows, cols = perm[r0:r1], perm[c0:c1]
        u, _ = aca.aca(lambda i: op.block(rows[[i]], cols)[0],
                       lambda j: op.block(rows, cols[[j]])[:, 0], r1 - r0, c1 - c0, eps, 64)
        pick = rng.choice(r1 - r0, min(64, r1 - r0), replace=False)
        A = op.block(rows[pick], cols)
        U, W = H.lr_factors(b)
        err = np.linalg.norm(A - U[pick] @ W.T) / np.linalg.norm(A)
        say("aca bins", precision, eps, (r1 - r0, c1 - c0), int(rank), u.shape[1], err)
        assert int(rank) >= u.shape[1] - 1
        if precision == "f64" or eps > 1e-5:
            assert int(rank) <= u.shape[1] + 1
        assert err <= 10 * eps
    H.free()
