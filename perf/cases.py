"""Timed cases of the H-matrix library: what a boundary-element program has it do.

Four kinds of pass, each through the package's public calls:

  build     an H-matrix from a mesh in host memory, one product with it, free
  product   H x or H^T x with a handle that the program keeps
  solve     GMRES, refined GMRES or CG on a kept handle
  adjoint   a differentiable solve: density, objective, gradient

The surfaces are radially perturbed, rotated geodesic spheres of 20 f^2 flat
triangles, less a few ("drop") for odd sizes and an open surface: the sizes and the
smooth shapes of the benchmark and the tests, without their exact symmetry.  Vectors
have the type that the benchmark gives each storage form: double for f64, float for
f32 and f16.  The forms keep the benchmark's tolerances (eps 1e-6, 1e-4 with f16
factors)."""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1806_11558_amd as hm

DEV = "cuda"


# ---------------------------------------------------------------- cases
def _case(name, kind, f, **kw):
    c = dict(name=name, kind=kind, f=f, drop=0, ngeom=1, form="f64", leaf=32, eps=1e-6,
             nrhs=1, transpose=False, operator="collocation", method="gmres", tol=1e-8)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call in use: the README's defaults on a test-sized mesh, one
        # product of a program's own iteration
        _case("product_f64_1k", "product", 8),
        # the transposed product of an adjoint on a small mesh of odd size, three columns
        _case("product_t_f32_20k_3rhs", "product", 32, drop=3, form="f32", nrhs=3,
              transpose=True),
        # an ordinary product: the benchmark's form at the size of its smaller workloads
        _case("product_f32_82k", "product", 64, form="f32", leaf=64),
        # sixteen right-hand sides at once, as the benchmark times them, in double
        _case("product_f64_82k_16rhs", "product", 64, leaf=64, nrhs=16),
        # many right-hand sides with 16-bit factors on a size that is no power of two
        _case("product_f16_162k_16rhs", "product", 90, drop=1, form="f16", leaf=64, eps=1e-4,
              nrhs=16),
        # the largest product of which several handles fit the card at once
        _case("product_f32_655k", "product", 181, form="f32", leaf=64),
        # a new small geometry in a design loop: set up with defaults and applied once
        _case("build_f64_1k", "build", 8),
        # many small geometries set up in one call, eight columns applied to all
        _case("build_batch12_f32", "build", 16, ngeom=12, form="f32", leaf=64, eps=1e-5, nrhs=8),
        # the largest setup: the benchmark's first headline figure, at a size of which a
        # few handles fit the card at once
        _case("build_f32_512k", "build", 160, form="f32", leaf=64),
        # the paper's own discretisation on an ordinary mesh
        _case("build_galerkin_f32_82k", "build", 64, form="f32", leaf=64, operator="galerkin"),
        # the whole solve of an ordinary mesh: refinement around float GMRES to 1e-8
        _case("solve_f32_refine_20k", "solve", 32, form="f32", leaf=64, method="refine"),
        # a differentiable solve of a small mesh: forward, objective, adjoint solve
        _case("adjoint_f64_5k", "adjoint", 16, tol=1e-10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the form, mesh size, leaf size, column count, direction and solver
    vary together; no case costs more than the largest listed ones (the product at
    655,000 and the build at 512,000 unknowns)."""
    kind = rng.choices(["product", "build", "solve", "adjoint"], weights=[5, 4, 2, 1])[0]
    form = rng.choices(["f64", "f32", "f16"], weights=[3, 4, 2])[0]
    leaf = rng.choice([24, 32, 32, 40, 50, 64, 64, 64])
    c = dict(kind=kind, form=form, leaf=leaf, drop=rng.randrange(0, 8), ngeom=1,
             nrhs=1, transpose=False, operator="collocation", method="gmres", tol=1e-8)
    c["eps"] = 1e-4 if form == "f16" else rng.choice([1e-6, 1e-6, 1e-5])
    if kind == "product":
        c["nrhs"] = rng.choices([1, 2, 3, 4, 5, 8, 11, 16, 24], weights=[8, 2, 2, 2, 1, 2, 1, 3, 1])[0]
        c["transpose"] = rng.random() < 0.3
        c["f"] = _log_int(rng, 5, 110 if form != "f64" else 70)
    elif kind == "build":
        c["operator"] = "galerkin" if rng.random() < 0.25 else "collocation"
        c["nrhs"] = rng.choice([1, 1, 4, 8])
        if rng.random() < 0.25:
            c["ngeom"] = rng.randint(2, 16)
        top = 48 if c["operator"] == "galerkin" else (110 if form != "f64" else 70)
        c["f"] = _log_int(rng, 5, max(6, int(top / math.sqrt(c["ngeom"]))))
    elif kind == "solve":
        if rng.random() < 0.3:
            c["operator"], c["method"], c["form"] = "galerkin", "cg", "f32"
            c["eps"] = 1e-6
        elif form != "f64":
            c["method"] = "refine"
        else:
            c["method"] = rng.choice(["gmres", "graph"])
            c["transpose"] = rng.random() < 0.3
        c["nrhs"] = rng.choice([1, 1, 2, 4, 8])
        c["f"] = _log_int(rng, 5, 40)
    else:
        c["form"], c["eps"], c["tol"] = "f64", 1e-6, 1e-10
        c["f"] = _log_int(rng, 5, 24)
    return c


# ---------------------------------------------------------------- meshes
@functools.lru_cache(maxsize=None)
def _geodesic(f):
    """Vertices on the unit sphere and the 20 f^2 triangles of the icosahedron whose
    faces are cut into f^2 pieces each; neighbours share vertex indices."""
    p = (1.0 + math.sqrt(5.0)) / 2.0
    v = np.array([[-1, p, 0], [1, p, 0], [-1, -p, 0], [1, -p, 0], [0, -1, p], [0, 1, p],
                  [0, -1, -p], [0, 1, -p], [p, 0, -1], [p, 0, 1], [-p, 0, -1], [-p, 0, 1]])
    faces = np.array([[0, 11, 5], [0, 5, 1], [0, 1, 7], [0, 7, 10], [0, 10, 11], [1, 5, 9],
                      [5, 11, 4], [11, 10, 2], [10, 7, 6], [7, 1, 8], [3, 9, 4], [3, 4, 2],
                      [3, 2, 6], [3, 6, 8], [3, 8, 9], [4, 9, 5], [2, 4, 11], [6, 2, 10],
                      [8, 6, 7], [9, 8, 1]])
    i, j = (a.ravel() for a in np.meshgrid(np.arange(f + 1), np.arange(f + 1), indexing="ij"))
    keep = i + j <= f
    i, j = i[keep], j[keep]                    # barycentric grid points of one face
    at = np.full((f + 2, f + 2), -1, dtype=np.int64)
    at[i, j] = np.arange(i.size)
    up = at[:f, :f].ravel() >= 0
    up &= (np.add.outer(np.arange(f), np.arange(f)).ravel() < f)
    a, b = np.divmod(np.nonzero(up)[0], f)
    tri = [np.stack([at[a, b], at[a + 1, b], at[a, b + 1]], 1)]
    dn = a + b < f - 1
    a, b = a[dn], b[dn]
    tri.append(np.stack([at[a + 1, b], at[a + 1, b + 1], at[a, b + 1]], 1))
    tri = np.concatenate(tri)
    # a point is named by its weights on the icosahedron's corners, at most three of them
    names, pts = [], []
    for q in faces:
        wgt = np.stack([f - i - j, i, j], 1).astype(np.int64)
        order = np.argsort(q)
        corner, wgt = q[order], wgt[:, order]
        # corners without weight leave no trace: shift the used ones together
        used = wgt > 0
        key = np.zeros((i.size, 3), dtype=np.int64)
        slot = np.cumsum(used, 1) - 1
        for k in range(3):
            r = np.nonzero(used[:, k])[0]
            key[r, slot[r, k]] = corner[k] * (f + 1) + wgt[r, k]
        base = 13 * (f + 1)
        names.append((key[:, 0] * base + key[:, 1]) * base + key[:, 2])
        pts.append(wgt @ v[corner] / f)
    names, pts = np.concatenate(names), np.concatenate(pts)
    _, first, inv = np.unique(names, return_index=True, return_inverse=True)
    V = pts[first]
    V /= np.linalg.norm(V, axis=1, keepdims=True)
    n1 = i.size
    T = np.concatenate([inv.reshape(-1)[k * n1:(k + 1) * n1][tri] for k in range(20)])
    return np.ascontiguousarray(V), np.ascontiguousarray(T.astype(np.int32))


def _mesh(f, drop, seed):
    """The geodesic sphere, radially perturbed by five seeded smooth waves and rotated."""
    V, T = _geodesic(f)
    g = np.random.default_rng(seed)
    r = np.ones(V.shape[0])
    for _ in range(5):
        r += 0.03 * np.cos(V @ g.normal(scale=1.5, size=3) + g.uniform(0, 2 * np.pi))
    q, _ = np.linalg.qr(g.normal(size=(3, 3)))
    q[:, 0] *= np.sign(np.linalg.det(q))       # a rotation: triangles keep their outside
    V = (V * r[:, None]) @ q.T
    return np.ascontiguousarray(V), np.ascontiguousarray(T[:T.shape[0] - drop])


def _meshes(case, seed):
    return [_mesh(case["f"], case["drop"], [seed, k]) for k in range(case["ngeom"])]


def _vectors(case, n, seed):
    """N(0,1) columns, as the benchmark's products and right-hand sides."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    shape = (n,) if case["nrhs"] == 1 else (n, case["nrhs"])
    x = torch.randn(shape, generator=g, dtype=torch.float64, device=DEV)
    return x if case["form"] == "f64" else x.float()


# ---------------------------------------------------------------- passes
def _build(case, meshes):
    kw = dict(leaf_size=case["leaf"], eta=1.0, eps=case["eps"], precision=case["form"],
              operator=case["operator"])
    if len(meshes) == 1:
        return hm.HMatrix(*meshes[0], **kw)
    return hm.HMatrix.batch(meshes, **kw)


def prepare(case, seed):
    # a program that goes on to another problem hands the last one's cached memory back:
    # the library keeps it otherwise, and meshes of changing sizes fill the card with it
    hm.release_memory()
    meshes = _meshes(case, seed)
    n = sum(t.shape[0] for _, t in meshes)
    state = {"case": case, "x": _vectors(case, n, seed)}
    if case["kind"] == "build":
        state["meshes"] = meshes
    else:
        state["H"] = _build(case, meshes)
    if case["kind"] == "adjoint":
        state["goal"] = _vectors(case, n, seed + (1 << 40))
    if case["kind"] == "product":
        state["y"] = torch.empty_like(state["x"])
    return state


def run(state):
    case, x = state["case"], state["x"]
    if case["kind"] == "build":
        H = _build(case, state["meshes"])
        y = H.matvec(x)
        H.free()
        return y
    H = state["H"]
    if case["kind"] == "product":
        return H.matvec(x, out=state["y"], transpose=case["transpose"])
    if case["kind"] == "solve":
        m = case["method"]
        s, info, status = H.solve(x, tol=case["tol"], max_iter=3000, transpose=case["transpose"],
                                  graph=m == "graph", refine=m == "refine",
                                  method="cg" if m == "cg" else "gmres")
        return s
    f = x.clone().requires_grad_(True)
    sigma = hm.hsolve(f, H, case["tol"])
    (0.5 * (sigma - state["goal"]).square().sum()).backward()
    return {"sigma": sigma.detach(), "grad": f.grad}


# ---------------------------------------------------------------- work
_STEPS = {"gmres": 60, "graph": 60, "refine": 75, "cg": 90}


def work(case):
    """From the stored entries per unknown, by fits to built matrices: the dense blocks
    hold the width of about 58 leaves, the factors about 129 columns of the average rank
    per tree level."""
    n1 = 20 * case["f"] ** 2 - case["drop"]
    n, leaf = n1 * case["ngeom"], case["leaf"]
    width = n1 / 2 ** math.ceil(math.log2(max(1.0, n1 / leaf)))     # rows of a leaf
    dense = n * min(n1, 58.0 * width)
    rank = {1e-4: 5.6, 1e-5: 7.2, 1e-6: 8.9}[case["eps"]]
    low = n * min(n1, 129.0 * rank * max(0.3, math.log2(n1 / (70.0 * width))))
    size = 8 if case["form"] == "f64" else 4
    held = size * dense + (2 if case["form"] == "f16" else size) * low
    vec = size * n * case["nrhs"]
    apply_b, apply_f = held + 2 * vec, 2.0 * (dense + low) * case["nrhs"]
    if case["kind"] == "product":
        return {"bytes": apply_b, "flops": apply_f}
    if case["kind"] == "build":
        per = 66 * (7 if case["operator"] == "galerkin" else 1)     # one kernel sum
        return {"bytes": held + 36.0 * n + 2 * vec, "flops": per * (dense + low) + apply_f}
    steps = 120 if case["kind"] == "adjoint" else _STEPS[case["method"]]
    return {"bytes": steps * apply_b, "flops": steps * apply_f}


# ---------------------------------------------------------------- 64-bit values
_S15 = math.sqrt(15.0)


def _nodes(V, T):
    """Radon's seven-point rule: nodes [7, n, 3], weights [7], areas, corners [n, 3, 3]."""
    P = torch.as_tensor(V, device=DEV)[torch.as_tensor(T.astype(np.int64), device=DEV)]
    c = P.mean(1)
    y = [c]
    for beta in ((1 + _S15) / 7, (1 - _S15) / 7):
        y += [c + beta * (P[:, k] - c) for k in range(3)]
    w = torch.tensor([9 / 40] + 3 * [(155 - _S15) / 1200] + 3 * [(155 + _S15) / 1200],
                     dtype=torch.float64)
    area = 0.5 * torch.linalg.cross(P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]).norm(dim=1)
    return torch.stack(y), w, area, P


def _inner(x, P):
    """int_T dy / |x - y| for points x [p, 3] and triangles P [p, 3, 3], in closed form
    over the three edges seen from x's projection on the triangle's plane."""
    nrm = torch.linalg.cross(P[:, 1] - P[:, 0], P[:, 2] - P[:, 0])
    nrm = nrm / nrm.norm(dim=1, keepdim=True)
    d = ((x - P[:, 0]) * nrm).sum(1)
    xp = x - d[:, None] * nrm
    d = d.abs()
    total = torch.zeros_like(d)
    for k in range(3):
        a, b = P[:, k], P[:, (k + 1) % 3]
        e = b - a
        le = e.norm(dim=1)
        t = e / le[:, None]
        cr = (torch.linalg.cross(a - xp, e) * nrm).sum(1)
        h = cr.abs() / le
        ok = h > 1e-14 * le
        h = torch.where(ok, h, torch.ones_like(h))
        la, lb = ((a - xp) * t).sum(1), ((b - xp) * t).sum(1)
        ra, rb = (x - a).norm(dim=1), (x - b).norm(dim=1)
        c = torch.sqrt(h * h + d * d)
        v = h * (torch.asinh(lb / c) - torch.asinh(la / c))
        v = v + d * (torch.atan(d * lb / (h * rb)) - torch.atan(d * la / (h * ra))
                     - torch.atan(lb / h) + torch.atan(la / h))
        total += torch.where(ok, torch.where(cr > 0, v, -v), torch.zeros_like(v))
    return total


def _touching(T):
    """All ordered pairs (i, j) of triangles that share a vertex, i = j among them."""
    n = T.shape[0]
    order = np.argsort(T.ravel(), kind="stable")
    vert, tri = T.ravel()[order], order // 3
    beg = np.searchsorted(vert, vert, "left")
    cnt = np.searchsorted(vert, vert, "right") - beg
    src = np.repeat(tri, cnt)
    off = np.arange(cnt.sum()) - np.repeat(np.cumsum(cnt) - cnt, cnt)
    dst = tri[np.repeat(beg, cnt) + off]
    return np.divmod(np.unique(src.astype(np.int64) * n + dst), n)


class _Dense:
    """Rows of the exact matrix of one mesh, in blocks."""

    def __init__(self, V, T, galerkin):
        self.y, self.w, self.area, P = _nodes(V, T)
        self.n, self.gal = T.shape[0], galerkin
        wa = self.area / (4 * math.pi)
        self.wa = wa
        if not galerkin:
            self.self_term = _inner(self.y[0], P) / (4 * math.pi)
            return
        i, j = _touching(T)
        self.i, self.j = (torch.as_tensor(a, device=DEV) for a in (i, j))
        g, gw = np.polynomial.legendre.leggauss(12)
        s, t = (a.ravel() for a in np.meshgrid(0.5 * (g + 1), 0.5 * (g + 1), indexing="ij"))
        q = (np.outer(gw, gw).ravel() / 4) * s
        self.val = torch.zeros(i.size, dtype=torch.float64, device=DEV)
        for b in range(0, i.size, 1 << 19):
            A, B = P[self.i[b:b + (1 << 19)]], P[self.j[b:b + (1 << 19)]]
            for k in range(s.size):
                x = A[:, 0] + s[k] * (A[:, 1] - A[:, 0]) + s[k] * t[k] * (A[:, 2] - A[:, 1])
                self.val[b:b + (1 << 19)] += q[k] * _inner(x, B)
        self.val *= 2 * self.area[self.i] / (4 * math.pi)

    def rows(self, b, e):
        out = torch.zeros(e - b, self.n, dtype=torch.float64, device=DEV)
        for p in range(7 if self.gal else 1):
            x = self.y[p, b:e]
            for q in range(7):
                d = self.y[q]
                r = (x[:, 0, None] - d[None, :, 0]).square_()
                r += (x[:, 1, None] - d[None, :, 1]).square_()
                r += (x[:, 2, None] - d[None, :, 2]).square_()
                out.add_(r.rsqrt_(), alpha=float(self.w[q] * (self.w[p] if self.gal else 1)))
        out *= self.wa[None, :]
        if not self.gal:
            k = torch.arange(b, e, device=DEV)
            out[k - b, k] = self.self_term[b:e]
            return out
        out *= self.area[b:e, None]
        m = (self.i >= b) & (self.i < e)
        out[self.i[m] - b, self.j[m]] = self.val[m]
        return out

    def blocks(self):
        step = max(1, int(1.5e8) // self.n)
        for b in range(0, self.n, step):
            yield b, min(self.n, b + step), self.rows(b, min(self.n, b + step))


def _apply(case, meshes, x):
    y = torch.zeros_like(x)
    at = 0
    for V, T in meshes:
        A = _Dense(V, T, case["operator"] == "galerkin")
        xs, ys = x[at:at + A.n], y[at:at + A.n]
        for b, e, R in A.blocks():
            if case["transpose"]:
                ys += (R * xs[b:e, None]).sum(0) if x.dim() == 1 else R.t().contiguous() @ xs[b:e]
            else:
                ys[b:e] = R @ xs
        at += A.n
    return y


def exact(case, seed):
    """The same matrix in 64 bits without compression: the seven-point rule, the closed
    diagonal (Galerkin: 7 x 7 points, closed inner integrals for touching pairs)."""
    n1 = 20 * case["f"] ** 2 - case["drop"]
    pairs = case["ngeom"] * n1 * n1 * (7 if case["operator"] == "galerkin" else 1)
    whole = case["kind"] in ("solve", "adjoint")
    if pairs > 5e10 or (whole and n1 > 26000):
        return None
    meshes = _meshes(case, seed)
    x = _vectors(case, n1 * case["ngeom"], seed).double()
    if not whole:
        return _apply(case, meshes, x)
    D = _Dense(*meshes[0], case["operator"] == "galerkin")
    A = torch.cat([R for _, _, R in D.blocks()])
    cols = x.reshape(n1, -1)
    if case["kind"] == "solve":
        M = A.t().contiguous() if case["transpose"] else A
        return torch.linalg.solve(M, cols).reshape(x.shape)
    s = torch.linalg.solve(A, cols)
    goal = _vectors(case, n1, seed + (1 << 40)).reshape(n1, -1)
    return {"sigma": s.reshape(x.shape),
            "grad": torch.linalg.solve(A.t().contiguous(), s - goal).reshape(x.shape)}
