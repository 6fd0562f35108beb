"""Singular Galerkin entries of slices that list their touching pairs in parts."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_singular_entries_of_wide_slices():
    """N = 516 with leaf 64: sibling clusters of 64 and 65 triangles, so dense
    Galerkin slices of 64 x 65 entries list their touching pairs in two parts;
    every entry against the oracle within its singular tolerance of 1e-12."""
    import paper_1806_11558_amd as hm
    from oracle import galerkin
    from synthetic import icosphere
    V, T = icosphere(4)
    T = T[np.sort(np.random.default_rng(3).choice(T.shape[0], 516, replace=False))]
    op = galerkin.GalerkinOperator(V, T)
    A = op.dense()
    H = hm.HMatrix(V, T, leaf_size=64, eps=1e-6, precision="f64", operator="galerkin")
    perm, db, wide = H.perm(), H.dense_blocks(), 0
    for b, (r0, r1, c0, c1) in enumerate(db[:, :4]):
        wide += c1 - c0 > 64
        D = H.dense_entries(b, db)
        ref = A[np.ix_(perm[r0:r1], perm[c0:c1])]
        assert np.all(np.abs(D - ref) <= 1e-12 * np.abs(ref)), b
    H.free()
    assert wide > 0
