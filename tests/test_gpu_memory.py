"""Device memory of a handle against mem_limit_bytes."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import say


@pytest.mark.parametrize("level,leaf,form,kw,limit", [
    (0, 32, "f64", {}, 16744), (1, 32, "f32", {}, 99620), (3, 32, "f64", {}, 24387525),
    (3, 8, "f64", {}, 79255646), (4, 64, "f64", {}, 181458355), (5, 32, "f64", {}, 1423628063),
    (4, 64, "f16", {}, 95854606), (4, 32, "f64", {"autotune": True}, 217448188),
    (3, 32, "f64", {"operator": "galerkin"}, 24484001)])
def test_handle_fits_its_limit(level, leaf, form, kw, limit):
    """Icospheres of 20 to 20,480 triangles build within limits that hold the stored
    blocks, the factors at the ranks of the oracle and the product workspaces of 16
    columns, with little to spare: the least limits that were accepted when
    one-column products alone had work units and x had no copy per leaf."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere
    V, T = icosphere(level)
    say("memory", level, leaf, form, kw)
    H = hm.HMatrix(V, T, leaf_size=leaf, eps=1e-4 if form == "f16" else 1e-6, precision=form,
                   mem_limit_bytes=limit, **kw)
    assert H.stats()["device_bytes"] <= limit
    H.free()
    with pytest.raises(hm.HMError) as e:                # and a limit is a limit
        hm.HMatrix(V, T, leaf_size=leaf, eps=1e-4 if form == "f16" else 1e-6, precision=form,
                   mem_limit_bytes=limit // 2, **kw)
    assert e.value.status == hm.HM_ERR_OOM


def test_full_device_takes_back_cached_blocks():
    """A solve whose Krylov basis is larger than the device (327,680 unknowns, 256
    columns, 1,000 steps: 672 GB) fails, and the blocks that a freed handle left in
    the library's cache are on the device again; other handles go on."""
    import paper_1806_11558_amd as hm
    from synthetic import icosphere
    say("full device")
    H = hm.HMatrix(*icosphere(7), leaf_size=64, eps=1e-2, precision="f16")
    K = hm.HMatrix(*icosphere(5), leaf_size=32, eps=1e-6)
    held = K.stats()["device_bytes"]
    x = torch.ones(H.n, dtype=torch.float32, device="cuda:0")
    y = H.matvec(x)
    torch.cuda.synchronize()
    K.free()
    before = torch.cuda.mem_get_info()[0]
    f = torch.ones((H.n, 256), dtype=torch.float64, device="cuda:0")
    used = before - torch.cuda.mem_get_info()[0]
    with pytest.raises(hm.HMError) as e:
        H.solve(f, tol=1e-3, restart=1000)
    assert e.value.status == hm.HM_ERR_OOM
    assert torch.cuda.mem_get_info()[0] + used - before >= 0.9 * held
    assert torch.equal(H.matvec(x), y)
    H.free()
