"""Solves at the edges of what they accept: streams that end before the handle,
sizes at the limit of the fixed workspace, values that are not finite."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import rel2, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_graph_workspace_outlives_its_stream():
    """A graph solve on a stream that is destroyed before the handle is freed: the
    workspace (328 MB of basis vectors) goes back to the pool."""
    import paper_1806_11558_amd as hm
    from paper_1806_11558_amd import _binding
    from synthetic import icosphere, normal_columns
    V, T = icosphere(4)
    f = torch.tensor(normal_columns(len(T), 8, seed=3), device=DEV)
    L = _binding.lib()                                  # the HIP runtime it is linked to
    say("graph workspace and its stream")
    for _ in range(2):                                  # second time: everything is loaded
        torch.cuda.synchronize()
        hm.release_memory()
        before = torch.cuda.mem_get_info()[0]
        st = C.c_void_p()
        assert L.hipStreamCreate(C.byref(st)) == 0
        H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f64")
        _, info, status = H.solve(f, tol=1e-6, restart=1000, graph=True, stream=st.value)
        assert status == hm.HM_OK
        assert L.hipStreamDestroy(st) == 0
        H.free()
        hm.release_memory()
        after = torch.cuda.mem_get_info()[0]
    assert before - after < 64 << 20, (before, after)


@pytest.mark.parametrize("n,fits", [(9978, True), (9979, False)])
def test_largest_fixed_workspace(n, fits):
    """16 columns at restart 100: the largest system whose workspace
    (8 (restart + 7) n nrhs bytes, the partial sums of 2,048-row tiles and the small
    arrays) fits the 134,217,728 bytes of the fixed array, and one unknown more."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere, normal_columns
    V, T = icosphere(5)
    T = T[:n]
    say("fixed workspace", n)
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f64")
    f = torch.tensor(normal_columns(n, 16, seed=6), device=DEV)
    sp = hm.SolveParams(tol=1e-8, restart=100, max_iter=300, transpose=0, use_x0=0, flags=0,
                        refine=0, inner_tol=0.0)
    a, b = torch.empty_like(f), torch.empty_like(f)
    sta, ia = hm.hm_solve(H._h, f, a, sp)
    if fits:
        stb, ib = hm.hm_solve_noalloc(H._h, f, b, sp)
        assert sta == stb == hm.HM_OK and ia.iters == ib.iters
        assert torch.equal(a, b)
        assert rel2(H.matvec(b).cpu().numpy(), f.cpu().numpy()) <= 1.5e-8
    else:
        with pytest.raises(hm.HMError) as e:
            hm.hm_solve_noalloc(H._h, f, b, sp)
        assert e.value.status == hm.HM_ERR_ARG
    H.free()


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("refine", [False, True])
def test_first_guess_not_finite(graph, refine):
    """Three columns, the first guess of one is NaN: the others are solved, that one is
    not converged and costs no steps of its own."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere, normal_columns
    V, T = icosphere(2)
    say("NaN in the first guess", graph, refine)
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f32" if refine else "f64")
    f = torch.tensor(normal_columns(H.n, 3, seed=8), device=DEV)
    x0 = torch.zeros_like(f)
    _, ref, st = H.solve(f, tol=1e-8, restart=60, refine=refine, graph=graph, x0=x0)
    assert st == hm.HM_OK
    x0[7, 1] = float("nan")
    s, info, st = H.solve(f, tol=1e-8, restart=60, max_iter=1000, refine=refine, graph=graph, x0=x0)
    assert st == hm.HM_NOT_CONVERGED and info.converged == 2
    assert info.iters <= ref.iters + 2
    r = (f - H.matvec(s)).cpu().numpy()
    F = f.cpu().numpy()
    for c in (0, 2):
        assert np.linalg.norm(r[:, c]) <= 1.5e-8 * np.linalg.norm(F[:, c])
    H.free()


def test_product_not_finite():
    """A triangle given twice: the entries of the pair, 1 / 0, are infinite, so the
    first product is not finite.  The solve ends there, not converged."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere, normal_columns
    V, T = icosphere(2)
    T = np.concatenate([T, T[:1]])
    say("infinite entries")
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f64")
    f = torch.tensor(normal_columns(H.n, 2, seed=9), device=DEV)
    s, info, st = H.solve(f, tol=1e-8, max_iter=500)
    assert st == hm.HM_NOT_CONVERGED and info.converged == 0
    assert info.iters <= 2
    H.free()


@pytest.mark.parametrize("kw", [{}, {"graph": True}, {"refine": True}, {"method": "cg"}],
                         ids=["gmres", "graph", "refine", "cg"])
def test_right_hand_side_not_finite(kw):
    """A right-hand side with a NaN, alone and among finite ones (one of them zero):
    not converged, its relative residual NaN, the others solved."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere, normal_columns
    V, T = icosphere(2)
    say("NaN in f", kw)
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-8, precision="f64",
                   operator="galerkin" if "method" in kw else "collocation")
    F = normal_columns(H.n, 3, seed=10)
    F[:, 2] = 0.0
    f = torch.tensor(F, device=DEV)
    _, ref, st = H.solve(f, tol=1e-8, **kw)
    assert st == hm.HM_OK
    f[5, 1] = float("nan")
    s, info, st = H.solve(f, tol=1e-8, **kw)
    assert st == hm.HM_NOT_CONVERGED and info.converged == 2
    assert np.isnan(info.rel_residual) and info.iters <= ref.iters + 2
    r = (f - H.matvec(s)).cpu().numpy()
    assert np.linalg.norm(r[:, 0]) <= 1.5e-8 * np.linalg.norm(F[:, 0])
    assert torch.count_nonzero(s[:, 2]).item() == 0
    s, info, st = H.solve(f[:, 1].contiguous(), tol=1e-8, **kw)
    assert st == hm.HM_NOT_CONVERGED and info.converged == 0
    assert np.isnan(info.rel_residual)
    H.free()


def test_adjoint_of_nan_raises():
    """A density from a right-hand side that is not finite is not handed on."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere
    V, T = icosphere(1)
    say("hsolve of NaN")
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f64")
    f = torch.ones(H.n, dtype=torch.float64, device=DEV)
    f[0] = float("nan")
    with pytest.raises(hm.HMError):
        hm.hsolve(f, H)
    H.free()


@pytest.mark.parametrize("level,counts", [(0, (3, 16, 17, 24, 63, 65, 100, 200)),
                                          (1, (5, 15, 17, 33, 40, 96, 129)), (2, (6, 24, 48, 70))])
@pytest.mark.parametrize("graph", [False, True])
def test_any_number_of_columns(level, counts, graph):
    """Columns in groups of up to 64 with as many rows at once as fit, below and above
    the 16 columns up to which the sums are folded: the residual of every column by the
    oracle's dense matrix, within the tolerance and 100 ACA eps; every column takes
    the values it has in a call of its own (to 1e-8, both solves end at 1e-10)."""
    import paper_1806_11558_amd as hm
    from oracle import bem
    from synthetic import icosphere, normal_columns
    V, T = icosphere(level)
    n = len(T)
    say("columns", level, graph)
    H = hm.HMatrix(V, T, leaf_size=32, eps=1e-10)
    A = bem.Operator(V, T).cols(np.arange(n))
    F = normal_columns(n, max(counts), seed=8)
    for nrhs in counts:
        f = torch.tensor(F[:, :nrhs].copy(), device=DEV)
        s, info, status = H.solve(f, tol=1e-10, graph=graph)
        assert status == hm.HM_OK and info.converged == nrhs
        x = s.cpu().numpy()
        for c in range(nrhs):
            assert np.linalg.norm(A @ x[:, c] - F[:, c]) <= 1.1e-8 * np.linalg.norm(F[:, c]), (nrhs, c)
        one, _, _ = H.solve(f[:, nrhs - 1:].contiguous(), tol=1e-10, graph=graph)
        assert rel2(one.cpu().numpy()[:, 0], x[:, nrhs - 1]) <= 1e-8
    H.free()
