"""Products whose column count fills no pass exactly, over every remainder of
the leaf size: the padded passes of 4, 8 and 16 columns, the row tiles of 16, 8
and 4 rows of the matrix-core phase 1 and the 1 to 4 row tiles of phase 2."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import rel2, say

DEV = "cuda:0"


@pytest.mark.parametrize("ld", [4, 8, 12, 16, 20, 28, 36, 44, 52, 60, 64])
@pytest.mark.parametrize("prec,eps", [("f64", 1e-8), ("f32", 1e-6), ("f16", 1e-4)])
def test_padded_passes_every_leaf_remainder(ld, prec, eps):
    """16 leaves of ld rows, and the same mesh without its last nine triangles
    (ragged leaves), 3, 5 and 11 columns in both directions against the dense
    oracle within 10 eps (plus the float accumulation of float vectors).  A
    column of NaN stays in its own column."""
    import paper_1806_11558_amd as hm
    from oracle import bem
    from synthetic import icosphere, normal_columns
    V, T = icosphere(3)
    for n in (16 * ld, 16 * ld - 9):
        say("passes", ld, prec, n)
        op = bem.Operator(V, T[:n])
        A = op.dense()
        H = hm.HMatrix(V, T[:n], leaf_size=ld, eps=eps, precision=prec)
        assert int(H.leaves()[:, 2].max()) == ld
        for vdt in ((torch.float64,) if prec == "f64" else (torch.float64, torch.float32)):
            bound = 10 * eps + (1e-6 if vdt == torch.float32 else 0.0)
            for nrhs in (3, 5, 11):
                x = normal_columns(n, nrhs, seed=nrhs)
                xt = torch.tensor(x, dtype=vdt, device=DEV)
                xt[:, 1] = float("nan")
                for ref, y in ((A @ x, H.matvec(xt)), (A.T @ x, H.matvec_T(xt))):
                    y = y.double().cpu().numpy()
                    assert np.isnan(y[:, 1]).all()
                    for k in range(nrhs):
                        if k != 1:
                            assert rel2(y[:, k], ref[:, k]) <= bound, (n, nrhs, k, vdt)
        H.free()


@pytest.mark.parametrize("leaves,ld", [(16, 4), (16, 12), (16, 20), (16, 36), (16, 52), (16, 64),
                                       (128, 12), (128, 24), (256, 12)])
@pytest.mark.parametrize("prec,eps", [("f64", 1e-8), ("f32", 1e-6), ("f16", 1e-4)])
def test_one_and_two_columns_by_tree_size(leaves, ld, prec, eps):
    """Trees of full and of ragged leaves on both sides of the size from which
    transposed products of one and two columns leave the matrix cores, both
    directions against the dense oracle within 10 eps (plus the float
    accumulation of float vectors); a column of NaN stays in its own column."""
    import paper_1806_11558_amd as hm
    from oracle import bem
    from synthetic import icosphere, normal_columns
    V, T = icosphere(4)
    for n in (leaves * ld, leaves * ld - 9):
        say("passes 1 2", leaves, ld, prec, n)
        A = bem.Operator(V, T[:n]).dense()
        H = hm.HMatrix(V, T[:n], leaf_size=ld, eps=eps, precision=prec)
        assert len(H.leaves()) == leaves
        for vdt in ((torch.float64,) if prec == "f64" else (torch.float64, torch.float32)):
            bound = 10 * eps + (1e-6 if vdt == torch.float32 else 0.0)
            x = normal_columns(n, 2, seed=5)
            x2 = torch.tensor(x, dtype=vdt, device=DEV)
            x1 = x2[:, 0].contiguous()
            for ref, f in ((A @ x, H.matvec), (A.T @ x, H.matvec_T)):
                assert rel2(f(x1).double().cpu().numpy(), ref[:, 0]) <= bound
                y = f(x2).double().cpu().numpy()
                for k in range(2):
                    assert rel2(y[:, k], ref[:, k]) <= bound, (n, k, vdt)
                xn = x2.clone()
                xn[:, 1] = float("nan")
                y = f(xn).double().cpu().numpy()
                assert np.isnan(y[:, 1]).all() and rel2(y[:, 0], ref[:, 0]) <= bound
        H.free()
