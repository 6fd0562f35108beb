"""GMRES over the forms of its orthogonalisation: column counts that are and are
not powers of two, more than a pinned page of results holds, tile sums folded
into the kernels or added by one of their own, two threads per row or one, and
the coarse row tiles of a fixed workspace that only they fit."""
import numpy as np
import pytest
import torch

from gpu_util import rel2, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("level,nrhs", [(1, 1), (3, 1), (3, 2), (3, 5), (3, 8), (3, 21), (2, 64),
                                        (2, 70), (4, 1), (4, 16)])
@pytest.mark.parametrize("refine", [False, True])
def test_gmres_column_counts(level, nrhs, refine):
    """N = 80 to 5,120, restart 25 (several cycles), residual 1e-10 by an
    independent double product of the same matrix."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere, normal_columns
    V, T = icosphere(level)
    say("arnoldi", level, nrhs, refine)
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f32" if refine else "f64")
    F = normal_columns(H.n, nrhs, seed=nrhs)
    if nrhs > 2:
        F[:, 1] = 0.0                                  # a zero column, and ...
        F[:, 2] *= 1e-9                                # ... one of another size
    f = torch.tensor(F[:, 0] if nrhs == 1 else F, device=DEV)
    s, info, st = H.solve(f, tol=1e-10, restart=25, refine=refine)
    assert st == hm.HM_OK and info.converged == nrhs
    r = (f - H.matvec(s)).cpu().numpy().reshape(H.n, -1)
    for c in range(nrhs):
        assert np.linalg.norm(r[:, c]) <= 1.5e-10 * np.linalg.norm(F[:, c]), c
    if nrhs > 2:
        assert torch.count_nonzero(s[:, 1]).item() == 0
    # steps ahead of the host change nothing: one column alone, bitwise
    if nrhs == 1:
        s2, info2, _ = H.solve(f, tol=1e-10, restart=25, refine=refine, graph=True)
        assert info2.iters == info.iters and torch.equal(s, s2)
    H.free()


def test_fixed_workspace_coarse_tiles():
    """64 columns, restart 196 at N = 1,280: 132 of the 134 MB of the fixed
    workspace are basis vectors, the fine tiles' partial sums no longer fit.
    hm_solve takes the same tiles: bitwise the same result."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere, normal_columns
    V, T = icosphere(3)
    say("coarse tiles")
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f64")
    f = torch.tensor(normal_columns(H.n, 64, seed=5), device=DEV)
    sp = hm.SolveParams(tol=1e-10, restart=196, max_iter=400, transpose=0, use_x0=0, flags=0,
                        refine=0, inner_tol=0.0)
    a, b = torch.empty_like(f), torch.empty_like(f)
    sta, ia = hm.hm_solve(H._h, f, a, sp)
    stb, ib = hm.hm_solve_noalloc(H._h, f, b, sp)
    assert sta == stb == hm.HM_OK and ia.iters == ib.iters
    assert torch.equal(a, b)
    assert rel2(H.matvec(b).cpu().numpy(), f.cpu().numpy()) <= 1.5e-10
    H.free()
