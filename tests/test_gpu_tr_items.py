"""Transposed products by the width of their V items: trees whose leaves differ
in padded size, where a block's factor is an item of its own as wide as its rank,
and trees of one size with items of up to 64 columns, on both sides of the leaf
counts from which four single-precision columns run on the vector units."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import rel2, say

DEV = "cuda:0"


@pytest.mark.parametrize("n,leaf,leaves,sizes", [
    (1100, 5, 256, (4, 8)), (2250, 5, 512, (4, 8)), (4500, 5, 1024, (4, 8)),
    (3200, 13, 256, (12, 16)), (12800, 13, 1024, (12, 16)),
    (4096, 4, 1024, (4,)), (8192, 4, 2048, (4,)), (8183, 4, 2048, (4,)), (16384, 8, 2048, (8,))])
@pytest.mark.parametrize("prec,eps", [("f64", 1e-8), ("f32", 1e-6), ("f16", 1e-4)])
def test_transposed_by_item_width(n, leaf, leaves, sizes, prec, eps):
    """1, 2, 3, 4 and 7 columns against 96 exact columns of the oracle within 10 eps
    (plus the float accumulation of float vectors); a column of NaN stays in its own
    column."""
    import paper_1806_11558_amd as hm
    from oracle import bem
    from synthetic import icosphere, normal_columns
    V, T = icosphere(5)
    T = T[:n]
    say("tr items", n, leaf, prec)
    H = hm.HMatrix(V, T, leaf_size=leaf, eps=eps, precision=prec)
    m = H.leaves()[:, 2]
    assert len(m) == leaves and set((m + 3) // 4 * 4) == set(sizes)
    pick = np.random.default_rng(1).choice(n, 96, replace=False)
    B = bem.Operator(V, T).cols(pick)
    x = normal_columns(n, 7, seed=4)
    ref = B.T @ x
    for vdt in ((torch.float64,) if prec == "f64" else (torch.float64, torch.float32)):
        bound = 10 * eps + (1e-6 if vdt == torch.float32 else 0.0)
        for nrhs in (1, 2, 3, 4, 7):
            xt = torch.tensor(x[:, :nrhs].copy(), dtype=vdt, device=DEV)
            y = H.matvec_T(xt).double().cpu().numpy()[pick]
            for k in range(nrhs):
                assert rel2(y[:, k], ref[:, k]) <= bound, (nrhs, k, vdt)
            if nrhs > 1:
                xt[:, 1] = float("nan")
                y = H.matvec_T(xt).double().cpu().numpy()[pick]
                assert np.isnan(y[:, 1]).all()
                for k in range(nrhs):
                    assert k == 1 or rel2(y[:, k], ref[:, k]) <= bound, (nrhs, k, vdt)
    H.free()


@pytest.mark.parametrize("n,leaf,leaves", [
    (500, 32, 16), (520, 32, 24), (1280, 64, 32), (1280, 24, 64), (2199, 64, 64),
    (2200, 64, 64), (2560, 24, 128)])
@pytest.mark.parametrize("prec,eps", [("f32", 1e-6), ("f16", 1e-4)])
def test_one_double_column_narrow_factors(n, leaf, leaves, prec, eps):
    """One and two double columns over narrower factors, on both sides of the sizes
    at which they move between the vector and the matrix units: within 10 eps
    of 96 exact columns of the oracle."""
    import paper_1806_11558_amd as hm
    from oracle import bem
    from synthetic import icosphere, normal_columns
    V, T = icosphere(4)
    T = T[:n]
    say("one column", n, leaf, prec)
    H = hm.HMatrix(V, T, leaf_size=leaf, eps=eps, precision=prec)
    assert len(H.leaves()) == leaves
    pick = np.random.default_rng(1).choice(n, 96, replace=False)
    B = bem.Operator(V, T).cols(pick)
    x = normal_columns(n, 2, seed=5)
    ref = B.T @ x
    for nrhs in (1, 2):
        y = H.matvec_T(torch.tensor(x[:, :nrhs].copy(), device=DEV)).cpu().numpy()[pick]
        for k in range(nrhs):
            assert rel2(y[:, k], ref[:, k]) <= 10 * eps, (nrhs, k)
    H.free()


@pytest.mark.parametrize("n,leaf", [(20, 64), (21, 64), (22, 64), (63, 64), (77, 24), (80, 4), (127, 64)])
def test_small_trees_all_columns(n, leaf):
    """Trees with no or hardly any admissible block, where x per leaf with its rows
    padded is longer than x and the terms together: forward and transposed, 1 to 17
    columns, against the dense matrix of the oracle within 10 eps."""
    import paper_1806_11558_amd as hm
    from oracle import bem
    from synthetic import icosphere, normal_columns
    V, T = icosphere(2)
    T = T[:n]
    say("small trees", n, leaf)
    H = hm.HMatrix(V, T, leaf_size=leaf, eps=1e-8)
    B = bem.Operator(V, T).cols(np.arange(n))
    x = normal_columns(n, 17, seed=6)
    for M, tr in ((B, False), (B.T, True)):
        ref = M @ x
        for nrhs in (1, 2, 4, 8, 16, 17):
            y = H.matvec(torch.tensor(x[:, :nrhs].copy(), device=DEV), transpose=tr).cpu().numpy()
            for k in range(nrhs):
                assert rel2(y[:, k], ref[:, k]) <= 1e-7, (tr, nrhs, k)
    H.free()
