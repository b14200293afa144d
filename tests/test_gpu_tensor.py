"""The tensor form of the operator (boxes on tensor-product grids, any
spacings) at the edges of its wave tiles, and the meshes that must not take
it.  Its parity with the oracle's assembled operator at ordinary shapes is
in test_gpu_core.py, test_gpu_dirichlet.py, test_gpu_adjoint.py and
test_gpu_fullsize.py, whose boxes run in this form.

Reference here: the Kronecker products of the axes' exact 1-D matrices in
extended precision.  (On the thin cells below the oracle's Gauss-point
entries are themselves off by about u L / h, L the box length and h the
spacing: the Jacobian is a difference of coordinates.)

Bound per row i, with u = 1.1e-16: the product forms every entry from three
1-D factors (at most 3 roundings each) and adds at most 3 terms in each of
three stages, so its error is below 25 u B_i,
B_i = sum_j (|Kx| My Mz + Mx |Ky| Mz + Mx My |Kz| + m M + k |B| + k^2 Meta)_ij |x_j|
(the separated stiffness terms, not their possibly smaller sum); the wall and
absorption terms come from at most 8 elements each, below 35 u of the same
B_i.  Together 60 u B_i, taken as 7e-15 B_i; one misplaced or missing entry
errs by about B_i / 27.
"""
import sys

import numpy as np
import pytest

import workloads as W
from oracle import helmholtz as H

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FREQ = 170.0


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    import paper_2112_00087_amd as pkg
    assert torch.cuda.is_available()
    return pkg


def graded_box(nx, ny, nz, seed):
    """A box whose spacings vary by up to a factor of three along each axis."""
    rng = np.random.default_rng(seed)
    mesh = W.box_mesh(nx, ny, nz)
    for d in range(3):
        u = np.unique(mesh["xyz"][:, d])
        v = np.concatenate([[0.0], np.cumsum(rng.uniform(0.5, 1.5, u.size - 1))])
        v *= u[-1] / v[-1]
        mesh["xyz"][:, d] = v[np.searchsorted(u, mesh["xyz"][:, d])]
    if not mesh["bface_src"].any():
        mesh["bface_src"][[0, -1]] = 1
    return mesh


def _reference(mesh, beta, eta, k, m):
    """(A, B) of the docstring as dense arrays on the mesh's nodes, A complex
    extended precision; eta per element or None."""
    L = np.longdouble
    M, K, C = [], [], []
    for d in range(3):
        x = np.unique(mesh["xyz"][:, d]).astype(L)
        h = np.diff(x)
        n = x.size
        Md, Kd, Cd = np.zeros((n, n), L), np.zeros((n, n), L), np.zeros((n, n), np.clongdouble)
        for e in range(n - 1):
            for a in range(2):
                for b in range(2):
                    Md[e + a, e + b] += h[e] / (3 if a == b else 6)
                    Kd[e + a, e + b] += (1 if a == b else -1) / h[e]
        for side, at in ((0, 0), (1, n - 1)):
            if np.any(mesh["bface_tag"] == 2 * d + side):
                Cd[at, at] += 1j * L(k) * np.clongdouble(beta[2 * d + side])
        M.append(Md)
        K.append(Kd)
        C.append(Cd)
    kr = lambda z, y, x: np.kron(z, np.kron(y, x))  # noqa: E731
    A = (kr(M[2], M[1], K[0] + C[0]) + kr(M[2], K[1] + C[1], M[0]) + kr(K[2] + C[2], M[1], M[0]) -
         L(m) * kr(M[2], M[1], M[0]))
    B = (kr(M[2], M[1], abs(K[0]) + abs(C[0])) + kr(M[2], abs(K[1]) + abs(C[1]), M[0]) +
         kr(abs(K[2]) + abs(C[2]), M[1], M[0]) + L(m) * kr(M[2], M[1], M[0]))
    if eta is not None:
        ref = np.array([[2, 1], [1, 2]], L) / 6
        Me = np.kron(ref, np.kron(ref, ref))
        X = mesh["xyz"].astype(L)
        for e, v in enumerate(mesh["hex"]):
            vol = np.prod(X[v[7]] - X[v[0]])
            A[np.ix_(v, v)] += 1j * L(k) ** 2 * L(eta[e]) * vol * Me
            B[np.ix_(v, v)] += L(k) ** 2 * L(eta[e]) * vol * Me
    return A, B.astype(np.float64)


def _within(got, want, bound):
    """Largest error over its bound."""
    return float(np.max(np.abs(got - want).astype(np.float64) / np.maximum(bound, 1e-300)))


def _beta(rng):
    return rng.uniform(0, 0.05, 6) + 1j * rng.uniform(-0.01, 0.01, 6)


# around the wave's 62 nodes along x, its 2 lines and 2 planes, single cells, several blocks
SIZES = [(1, 1, 1), (2, 1, 3), (3, 4, 2), (60, 3, 4), (61, 2, 3), (62, 5, 2), (63, 2, 1), (123, 3, 3), (124, 4, 2),
         (20, 12, 10), (7, 40, 5), (5, 6, 41)]


@pytest.mark.parametrize("eta", [False, True])
@pytest.mark.parametrize("size", SIZES)
def test_product_and_diag(P, size, eta):
    say("tensor product", size, "eta" if eta else "")
    rng = np.random.default_rng(sum(size))
    mesh = graded_box(*size, seed=sum(size))
    beta = _beta(rng)
    e = rng.uniform(0, 0.02, mesh["n_elems"]) if eta else None
    for gls in (False, True):
        if eta and gls:
            continue
        S = H.System(mesh, beta, e, gls=gls)
        k = W.wavenumber(FREQ)
        A, B = _reference(mesh, beta, e, k, S.mass_coefficient(k))
        m = P.Helmholtz(mesh, beta, eta=e, gls=gls)
        m.set_frequency(FREQ)
        assert m.spmv_bytes("fp64", "tensor") == 32 * S.n + (8 * mesh["n_elems"] if eta else 0)
        x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
        y = m.apply(torch.as_tensor(x, device="cuda")).cpu().numpy()
        assert _within(y, A @ x, 7e-15 * (B @ np.abs(x))) <= 1.0
        d = m.diag().cpu().numpy()
        assert _within(d, A.diagonal(), 7e-15 * B.diagonal()) <= 1.0
        m.close()


@pytest.mark.parametrize("size", [(3, 4, 2), (62, 5, 2), (20, 12, 10)])
def test_missing_walls(P, size):
    """A box without the faces of two walls."""
    say("tensor missing walls", size)
    rng = np.random.default_rng(5 + sum(size))
    mesh = graded_box(*size, seed=sum(size))
    keep = ~np.isin(mesh["bface_tag"], (1, 2))
    for key in ("bface", "bface_tag", "bface_src"):
        mesh[key] = mesh[key][keep]
    beta = _beta(rng)
    k = W.wavenumber(FREQ)
    m = P.Helmholtz(mesh, beta)
    m.set_frequency(FREQ)
    assert m.spmv_bytes("fp64", "tensor") > 0
    A, B = _reference(mesh, beta, None, k, k * k)
    n = mesh["n_nodes"]
    x = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    y = m.apply(torch.as_tensor(x, device="cuda")).cpu().numpy()
    assert _within(y, A @ x, 7e-15 * (B @ np.abs(x))) <= 1.0
    m.close()


@pytest.mark.parametrize("what", ["moved-node", "two-tags", "face-twice", "shuffled-elements", "dirichlet"])
def test_other_meshes_keep_the_stored_forms(P, what):
    say("no tensor form:", what)
    rng = np.random.default_rng(3)
    mesh = graded_box(6, 5, 4, seed=1)
    beta = _beta(rng)
    if what == "moved-node":
        mid = W.node_id(3, 2, 2, 6, 5)
        mesh["xyz"][mid, 1] += 1e-9
    elif what == "two-tags":
        mesh["bface_tag"][0] = 3
    elif what == "face-twice":
        for key in ("bface", "bface_tag", "bface_src"):
            mesh[key] = np.concatenate([mesh[key], mesh[key][:1]])
    elif what == "shuffled-elements":
        mesh["hex"] = mesh["hex"][::-1].copy()
    S = H.System(mesh, beta, None, dirichlet=what == "dirichlet")
    m = P.Helmholtz(mesh, beta, dirichlet=what == "dirichlet")
    m.set_frequency(FREQ)
    with pytest.raises(P.HzError):
        m.spmv_bytes("fp64", "tensor")
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    A = S.operator(W.wavenumber(FREQ))
    y = m.apply(torch.as_tensor(x, device="cuda")).cpu().numpy()
    bound = 1e-14 * np.asarray(abs(A).sum(axis=1)).ravel() * np.abs(x).max()
    assert _within(y, A @ x, bound) <= 1.0
    m.close()


METHODS = [("gmres", dict(restart=40)), ("bicgstab", {}), ("bicgstabl", dict(restart=1)), ("bicgstabl", dict(restart=4)),
           ("bicgstabl", dict(restart=8)), ("tfqmr", {})]


@pytest.mark.parametrize("form", ["tensor", "stencil"])
@pytest.mark.parametrize("method,kw", METHODS)
def test_every_method_solves(P, monkeypatch, form, method, kw):
    """Each method in the tensor form (D^-1-scaled product inputs) and in the
    stencil form, from a non-zero start, in both precisions and without the
    preconditioner, against the oracle's direct solution: ||x - x*|| <=
    kappa tol with kappa below 1e3 at this size and frequency."""
    from oracle import direct
    say("solve", form, method, kw)
    monkeypatch.setenv("HZ_TENSOR", "1" if form == "tensor" else "0")
    rng = np.random.default_rng(11)
    mesh = graded_box(14, 9, 8, seed=2)
    for eta, dirichlet in ((False, False), (True, False), (True, True)):
        beta = _beta(rng)
        e = rng.uniform(0, 0.02, mesh["n_elems"]) if eta else None
        S = H.System(mesh, beta, e, dirichlet=dirichlet)
        k = W.wavenumber(90.0)
        g = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
        f = S.load(g, k)
        ref = direct.SparseLU(S.operator(k)).solve(f)
        m = P.Helmholtz(mesh, beta, eta=e, dirichlet=dirichlet)
        m.set_frequency(90.0)
        ft = torch.as_tensor(f, device="cuda")
        x0 = torch.as_tensor(1e-3 * g, device="cuda")
        for opts in (dict(), dict(precond="none"), dict(precision="mixed", inner_tol=1e-3)):
            if method == "gmres" and opts.get("precond") == "none":
                continue   # restarted GMRES stagnates without the scaling
            o = dict(method=method, tol=1e-10, max_matvec=40000, inner_restart=40, **kw, **opts)
            p, info = m.solve(ft, x0=x0, **o)
            err = np.linalg.norm(p.cpu().numpy() - ref) / np.linalg.norm(ref)
            say("  ", "eta" if eta else "", opts, info["status"], info["matvecs"], info["inner_matvecs"], f"{err:.1e}")
            assert info["status"] == 0 and err <= 1e-7
        m.close()


def test_changed_parameters_reach_every_path(P):
    """set_params on a tensor-form context: the product, the stored complex
    form (assembled on demand) and a sweep all see the new field."""
    rng = np.random.default_rng(21)
    mesh = graded_box(12, 8, 7, seed=4)
    beta = _beta(rng)
    m = P.Helmholtz(mesh, beta)
    e = rng.uniform(0, 0.02, mesh["n_elems"])
    m.set_params(_beta(rng), rng.uniform(0, 0.02, mesh["n_elems"]))
    m.set_params(beta, e)
    fresh = P.Helmholtz(mesh, beta, eta=e)
    x = torch.as_tensor(rng.standard_normal(m.n) + 1j * rng.standard_normal(m.n), device="cuda")
    for q in (m, fresh):
        q.set_frequency(FREQ)
    assert torch.equal(m.apply(x), fresh.apply(x))
    assert m.time_spmv(2, "fp64", "complex") > 0
    X = x[:, None].expand(-1, 3).contiguous()
    a, b = (q.apply_sweep([50.0, 100.0, 150.0], X)[0] for q in (m, fresh))
    assert float((a - b).norm() / b.norm()) < 1e-14
    with pytest.raises(P.HzError):
        m.set_params(beta, np.full(mesh["n_elems"], np.nan))
    m.close()
    fresh.close()


@pytest.mark.parametrize("method,kw", [("bicgstab", {}), ("bicgstabl", dict(restart=4)), ("tfqmr", {})])
def test_more_blocks_than_a_kernel_adds(P, monkeypatch, method, kw):
    """A plate of 4 x 401 x 401 nodes: 2,513 tiles of rows and 10,201 product
    blocks, so the sums are added by kernels of their own in both forms.  The
    iterates after 40 products agree: the two forms differ by rounding
    (1e-16), which 40 products far from convergence do not raise by 1e6."""
    say("many blocks:", method, kw)
    rng = np.random.default_rng(8)
    mesh = W.box_mesh(3, 400, 400)
    beta = _beta(rng)
    g = torch.as_tensor(rng.standard_normal(mesh["n_nodes"]) + 0j, device="cuda")
    x = {}
    for form in ("1", "0"):
        monkeypatch.setenv("HZ_TENSOR", form)
        m = P.Helmholtz(mesh, beta)
        m.set_frequency(60.0)
        x[form], info = m.solve(m.load(g), method=method, tol=1e-12, max_matvec=40, **kw)
        assert info["matvecs"] >= 32 and np.isfinite(info["relres_true"])
        m.close()
    assert float((x["1"] - x["0"]).norm() / x["0"].norm()) <= 1e-10


# columns around the lane groups (64 / s groups of 2 nodes along x, 4 waves a block: 8 nodes a
# block at 64 columns, 512 at one), odd sizes against the 2 x 2 patch, single cells
@pytest.mark.parametrize("eta", [False, True])
@pytest.mark.parametrize("size,nf", [((1, 1, 1), 64), ((8, 3, 4), 64), ((7, 4, 3), 33), ((16, 2, 5), 32),
                                     ((15, 6, 2), 13), ((33, 2, 2), 8), ((31, 3, 3), 3), ((20, 5, 4), 2),
                                     ((65, 2, 2), 1)])
def test_sweep_product(P, monkeypatch, size, nf, eta):
    """The multi-vector product in the tensor form, in one run of planes, in
    runs of two and as tuned.  complex64 vectors hold float32 inputs exactly,
    so their outputs carry one rounding (2^-24) beyond the FP64 bound."""
    say("tensor sweep product", size, nf, "eta" if eta else "")
    rng = np.random.default_rng(sum(size) + nf)
    mesh = graded_box(*size, seed=sum(size))
    beta = _beta(rng)
    e = rng.uniform(0, 0.02, mesh["n_elems"]) if eta else None
    S = H.System(mesh, beta, e, gls=not eta)
    m = P.Helmholtz(mesh, beta, eta=e, gls=not eta)
    freqs = np.linspace(60.0, 240.0, nf)
    x = (rng.standard_normal((S.n, nf)) + 1j * rng.standard_normal((S.n, nf))).astype(np.complex64)
    X = torch.as_tensor(x.astype(np.complex128), device="cuda")
    for chunks in (1, max(1, (size[2] + 1) // 2), None):
        if chunks:
            monkeypatch.setenv("HZ_SPMM_VARIANT", str(20000000 + chunks))
        else:
            monkeypatch.delenv("HZ_SPMM_VARIANT")
        for precision in ("fp64", "mixed"):
            Y, code = m.apply_sweep(freqs, X, precision=precision)
            assert code == 20000000 + chunks if chunks else code > 20000000
            for c in sorted({0, nf // 2, nf - 1}):
                k = W.wavenumber(freqs[c])
                A, B = _reference(mesh, beta, e, k, S.mass_coefficient(k))
                want = A @ x[:, c].astype(np.complex128)
                bound = 7e-15 * (B @ np.abs(x[:, c]))
                if precision == "mixed":
                    bound = bound + 2.0**-23 * np.abs(want).astype(np.float64)
                assert _within(Y[:, c].cpu().numpy(), want, bound) <= 1.0
    m.close()


# basis vectors per thread change at 16 and 32, the small-system kernels end at a restart
# length of 56 and at 16,384 rows (31x31x17 nodes are 16,337 rows in 64 tiles, 32x31x17 are 67)
@pytest.mark.parametrize("size,restart", [((2, 1, 1), 1), ((6, 5, 4), 3), ((9, 8, 7), 16), ((9, 8, 7), 17),
                                          ((9, 8, 7), 32), ((9, 8, 7), 33), ((9, 8, 7), 56), ((9, 8, 7), 57),
                                          ((30, 30, 16), 30), ((31, 30, 16), 30)])
def test_gmres_of_small_boxes(P, monkeypatch, size, restart):
    """One restart cycle and two: the residual estimate from the rotations is
    the true residual (Arnoldi identity, kept to 1e-10 by two Gram-Schmidt
    passes), the same in the stencil form, and no basis is read beyond the
    columns formed when the cap stops a cycle early."""
    say("small GMRES", size, restart)
    rng = np.random.default_rng(restart)
    mesh = graded_box(*size, seed=sum(size))
    beta = _beta(rng)
    g = torch.as_tensor(rng.standard_normal(mesh["n_nodes"]) + 1j * rng.standard_normal(mesh["n_nodes"]), device="cuda")
    for cap in (restart + 1, restart + 2 + restart // 2, 2 * restart + 2):
        res, x = [], []
        for form in ("1", "0"):
            monkeypatch.setenv("HZ_TENSOR", form)
            m = P.Helmholtz(mesh, beta)
            m.set_frequency(80.0)
            f = m.load(g)
            p, info = m.solve(f, method="gmres", restart=restart, tol=1e-12, max_matvec=cap)
            r = float((f - m.apply(p)).norm() / f.norm())
            assert info["matvecs"] <= cap + 1 and abs(info["relres_true"] - r) <= 1e-10
            res.append(r)
            x.append(p)
            m.close()
        assert abs(res[0] - res[1]) <= 1e-8 * max(res) + 1e-11
        assert float((x[0] - x[1]).norm()) <= 1e-7 * float(x[1].norm())


@pytest.mark.parametrize("parts,inner,eta,precision", [((2, 2, 1), "bicgstabl", False, "fp64"),
                                                       ((3, 1, 2), "gmres", True, "fp64"),
                                                       ((1, 2, 2), "tfqmr", False, "mixed"),
                                                       ((1, 1, 1), "bicgstab", False, "fp64")])
def test_schwarz_subdomains(P, monkeypatch, parts, inner, eta, precision):
    """Stacked subdomains of unequal sizes in the tensor form, their interface
    terms as corner entries, against the stored forms: the interface
    iterations are the same up to rounding, both glued solutions have a
    residual below 1e-8 (kappa below 1e2)."""
    say("tensor Schwarz", parts, inner, "eta" if eta else "", precision)
    rng = np.random.default_rng(sum(parts))
    mesh = W.box_mesh(14, 10, 8)
    beta = rng.uniform(0.005, 0.05, 6) + 1j * rng.uniform(-0.01, 0.01, 6)
    e = rng.uniform(0, 0.02, mesh["n_elems"]) if eta else None
    g = np.zeros(mesh["n_nodes"], complex)
    pn = W.patch_nodes(mesh)
    g[pn] = rng.standard_normal(pn.size) + 1j * rng.standard_normal(pn.size)
    x = []
    for form in ("1", "0"):
        monkeypatch.setenv("HZ_TENSOR", form)
        m = P.Helmholtz(mesh, beta, eta=e, parts=parts)
        m.set_frequency(90.0)
        p, info = m.solve(m.load(torch.as_tensor(g, device="cuda")), method="schwarz", restart=100, tol=1e-8,
                          max_matvec=1000, inner_tol=1e-11, dd_inner=inner, precision=precision,
                          inner_restart=4 if inner == "bicgstabl" else 30)
        say("  ", info["status"], info["iters"], info["inner_matvecs"], info["relres_true"])
        assert info["status"] == 0 and info["relres_true"] <= 1e-8
        x.append(p)
        m.close()
    assert float((x[0] - x[1]).norm()) <= 2e-6 * float(x[1].norm())


def test_apply_in_place(P):
    """y = A x into x itself and into a vector that overlaps x."""
    rng = np.random.default_rng(31)
    mesh = graded_box(20, 9, 8, seed=3)
    m = P.Helmholtz(mesh, _beta(rng))
    m.set_frequency(FREQ)
    buf = torch.as_tensor(rng.standard_normal(m.n + 5) + 1j * rng.standard_normal(m.n + 5), device="cuda")
    for x, y in ((slice(0, m.n), slice(0, m.n)), (slice(0, m.n), slice(5, m.n + 5)), (slice(5, m.n + 5), slice(0, m.n))):
        b = buf.clone()
        want = m.apply(b[x].clone())
        m.apply(b[x], out=b[y])
        assert torch.equal(torch.view_as_real(b[y]), torch.view_as_real(want))
    m.close()
