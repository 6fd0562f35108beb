"""The ACA's step kernels where their batches of terms end: ranks below and
above the eight terms whose dots ride on the residual row and above the
first pass's cap, in every kernel class, against the ACA of the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import say


@pytest.mark.parametrize("operator", ["collocation", "galerkin"])
@pytest.mark.parametrize("eps", [1e-3, 1e-6, 1e-11])
def test_ranks_and_factors_by_class(operator, eps):
    """Three blocks of every size bin (up to 64, 128, 256, 512, 1,024 and more
    rows) of N = 8,000 (leaf 48): the rank of the oracle's ACA on the exact
    block within one (equal pivots of the regular mesh may be taken in another
    order), the factors within 10 eps of it."""
    import paper_1806_11558_amd as hm
    from oracle import aca, bem, galerkin
    from synthetic import icosphere
    V, T = icosphere(5)
    T = T[:8000]
    op = (bem.Operator if operator == "collocation" else galerkin.GalerkinOperator)(V, T)
    H = hm.HMatrix(V, T, leaf_size=48, eta=2.0, eps=eps, max_rank=80, precision="f64",
                   operator=operator)
    lb, perm = H.lr_blocks(), H.perm()
    mx = np.maximum(lb[:, 1] - lb[:, 0], lb[:, 3] - lb[:, 2])
    rng, seen = np.random.default_rng(7), []
    for lo, hi in ((0, 64), (64, 128), (128, 256), (256, 512), (512, 1024), (1024, 1 << 30)):
        pool = np.flatnonzero((mx > lo) & (mx <= hi))
        for b in rng.choice(pool, min(3, pool.size), replace=False):
            r0, r1, c0, c1, rank, _ = lb[b]
            A = op.block(perm[r0:r1], perm[c0:c1])
            U, W = H.lr_factors(int(b))
            u, _ = aca.aca_dense(A, eps, 80)[:2]
            say("aca", operator, eps, A.shape, int(rank), u.shape[1])
            assert abs(int(rank) - u.shape[1]) <= 1
            assert np.linalg.norm(A - U @ W.T) <= 10 * eps * np.linalg.norm(A)
            seen.append(int(rank))
    H.free()
    assert eps > 1e-5 or max(seen) > 8
    assert eps > 1e-8 or max(seen) > 24
