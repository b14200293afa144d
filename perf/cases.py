"""What a user of this library has it do, as cases that can be timed and checked.

A user assembles a cavity mesh once (``Helmholtz``), then for every frequency
of interest forms the operator, loads the patch datum and solves; sweeps many
frequencies at once; differentiates a receiver energy; or splits the box into
subdomains.  The kinds below are those calls:

* ``product``   y = A(k) x with the formed operator (``apply``)
* ``solve``     set_frequency, load, solve: one frequency of one system
* ``sweep``     ``solve_sweep``: up to 64 frequencies advanced together
* ``gradient``  ``HelmholtzEnergy`` forward and backward over a few
  frequencies: J, dJ/dbeta per wall and dJ/deta per element
* ``schwarz``   set_frequency, load, solve by the Schwarz method

Meshes: the structured box of the cavity (``box``), its unstructured
hexahedral and tetrahedral meshes in random numbering (``hex``, ``tet``),
which a user gives to the library with RCM and length-sorted rows.  Solves
run to a relative residual of 1e-12 (the library's own tolerance for subdomain
solves): the accuracy a caller takes who differentiates or compares solutions,
and tight enough that every method's answer is the system's solution to about
ten digits.

``exact`` assembles the same discrete operator element by element in FP64
with torch and solves it directly: by the box's separable eigenvectors as the
preconditioner of a GMRES that is exact to rounding, or by a dense
factorisation where the mesh is small and unstructured.
"""
import math

import numpy as np
import torch

import workloads as W
from paper_2112_00087_amd import Helmholtz
from paper_2112_00087_amd.autograd import HelmholtzEnergy

TOL = 1e-12
DENSE = 5000          # nodes up to which exact() factorises a dense matrix
CAP = 60000           # products a solve may take


# ---------------------------------------------------------------- the cases
def _case(name, kind, mesh, nx, ny, nz, **more):
    c = dict(name=name, kind=kind, mesh=mesh, nx=nx, ny=ny, nz=nz, freq=100.0, nfreq=1, method="tfqmr", restart=4,
             precision="fp64", eta=False, gls=False, dirichlet=False)
    c.update(more)
    return c


def listed():
    return [
        # one product of the smallest mesh: what a caller's own iteration pays per call, all latency
        _case("product-box-20x12x10", "product", "box", 20, 12, 10),
        # one product of the largest cavity: all bandwidth
        _case("product-box-200x120x100", "product", "box", 200, 120, 100, freq=150.0),
        # the same on an unstructured tetrahedral mesh of ordinary size
        _case("product-tet-40x28x24", "product", "tet", 40, 28, 24, freq=180.0),
        # a small system end to end: launches and their gaps
        _case("solve-gmres30-box-20x12x10", "solve", "box", 20, 12, 10, method="gmres", restart=30),
        # the headline's method (BiCGStab) on the mesh of the sweep
        _case("solve-bicgstab-box-80x48x40", "solve", "box", 80, 48, 40, freq=90.0, method="bicgstab"),
        # the headline cavity and frequency with the method a user would pick there
        _case("solve-tfqmr-box-160x96x80", "solve", "box", 160, 96, 80, freq=250.0),
        # complex64 inner solves with FP64 refinement, odd sizes, stabilised scheme
        _case("solve-mixed-box-57x43x31", "solve", "box", 57, 43, 31, freq=140.0, precision="mixed", gls=True),
        # unstructured hexahedra, Dirichlet source, BiCGStab(4)
        _case("solve-bicgstabl-hex-9x7x6", "solve", "hex", 9, 7, 6, freq=120.0, method="bicgstabl", dirichlet=True),
        # the 64-frequency sweep
        _case("sweep-box-80x48x40-64", "sweep", "box", 80, 48, 40, nfreq=64),
        # a short sweep with a ragged column count and odd sizes
        _case("sweep-box-37x25x19-13", "sweep", "box", 37, 25, 19, nfreq=13, method="bicgstabl", restart=4),
        # gradient with an absorption field
        _case("gradient-box-40x24x20-4", "gradient", "box", 40, 24, 20, nfreq=4, method="bicgstabl", eta=True),
        # domain decomposition into 2 x 2 x 1 subdomains
        _case("schwarz-box-28x20x16", "schwarz", "box", 28, 20, 16, method="bicgstabl"),
    ]


def _box_size(rng, lo, hi):
    """Element counts of a cavity box with about n nodes, n log-uniform in lo..hi; each axis stretched by itself."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    h = (n / (1.8 * 1.2)) ** (1.0 / 3.0)
    return [max(3, round(h * s * rng.uniform(0.88, 1.12))) for s in (1.8, 1.2, 1.0)]


def draw(rng):
    kind = rng.choice(["product", "product", "solve", "solve", "solve", "sweep", "gradient", "schwarz"])
    mesh = "box"
    more = {}
    if kind == "product":
        mesh = rng.choice(["box", "box", "tet", "hex"])
        if mesh == "box":
            size = _box_size(rng, 3000, 2000000)
        else:
            size = _box_size(rng, 500, 20000 if mesh == "tet" else 900)
        more = dict(freq=round(rng.uniform(40.0, 250.0), 3), eta=rng.random() < 0.25, gls=rng.random() < 0.25)
    elif kind == "solve":
        mesh = rng.choice(["box", "box", "box", "tet"])
        size = _box_size(rng, 2500, 300000 if mesh == "box" else 12000)
        method = rng.choice(["bicgstab", "bicgstabl", "tfqmr", "tfqmr"])
        more = dict(freq=round(rng.uniform(60.0, 130.0), 3), method=method, restart=rng.choice([2, 4, 8]),
                    precision="mixed" if method == "tfqmr" and rng.random() < 0.4 else "fp64",
                    gls=rng.random() < 0.25, dirichlet=rng.random() < 0.25, eta=rng.random() < 0.15)
    elif kind == "sweep":
        size = _box_size(rng, 3000, 60000)
        method = rng.choice(["tfqmr", "tfqmr", "bicgstabl"])
        more = dict(nfreq=rng.randint(2, 64), method=method,
                    precision="mixed" if method == "tfqmr" and rng.random() < 0.3 else "fp64")
    elif kind == "gradient":
        size = _box_size(rng, 3000, 60000)
        more = dict(nfreq=rng.randint(1, 4), method=rng.choice(["tfqmr", "bicgstabl"]), eta=True)
    else:
        size = _box_size(rng, 2500, 12000)
        more = dict(freq=round(rng.uniform(60.0, 130.0), 3), method="bicgstabl")
    c = _case("", kind, mesh, *size, **more)
    del c["name"]
    return c


def _freqs(c):
    if c["nfreq"] == 1:
        return np.array([c["freq"]])
    return np.linspace(20.0, 300.0, c["nfreq"]) if c["kind"] == "sweep" else np.linspace(50.0, 150.0, c["nfreq"])


def _counts(c):
    """(nodes, elements) of the case's mesh."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    v, cells = (nx + 1) * (ny + 1) * (nz + 1), nx * ny * nz
    if c["mesh"] == "box":
        return v, cells
    if c["mesh"] == "tet":
        return v, 6 * cells
    rim = nx * ny + ny * nz + nx * nz
    edges = 7 * cells + 2 * rim + nx * ny + ny * nz + nx * nz + nx + ny + nz
    faces = 12 * cells + 2 * rim
    return v + edges + faces + 6 * cells, 24 * cells


def work(c):
    """Vectors in and out, each once: a right-hand side and a solution (or a product's x and y) per frequency; a
    gradient also reads the absorption field and writes its derivative.  The flops are one product's per frequency:
    how many products a solve needs is the data's affair."""
    n, ne = _counts(c)
    f = c["nfreq"]
    row = 15 if c["mesh"] == "tet" else 27
    b = 32 * n * f + (16 * ne if c["kind"] == "gradient" else 0)
    return {"bytes": b * (2 if c["kind"] == "gradient" else 1), "flops": 4 * row * n * f}


# ---------------------------------------------------------------- inputs
def _mesh(c, seed):
    size = (c["nx"], c["ny"], c["nz"])
    if c["mesh"] == "box":
        return W.box_mesh(*size)
    make = W.kuhn_tet_mesh if c["mesh"] == "tet" else W.kuhn_hex_mesh
    return make(*size, seed=seed)


def _inputs(c, seed):
    """Mesh, wall admittances, nodal patch values, absorption field, receivers and the product's vector."""
    rng = np.random.default_rng(seed)
    mesh = _mesh(c, seed)
    n, ne = mesh["n_nodes"], mesh["n_elems"]
    beta = rng.uniform(0.005, 0.05, 6) + 1j * rng.uniform(-0.01, 0.01, 6)
    g = np.zeros(n, dtype=np.complex128)
    pn = W.patch_nodes(mesh)
    g[pn] = rng.standard_normal(pn.size) + 1j * rng.standard_normal(pn.size)
    eta = rng.uniform(0.0, 0.02, ne) if c["eta"] else None
    rec = np.sort(rng.choice(n, size=min(16, n), replace=False))
    x = None
    if c["kind"] == "product":
        x = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    return mesh, beta, g, eta, rec, x


def _opts(c):
    o = dict(method=c["method"], restart=c["restart"], precision=c["precision"], tol=TOL, max_matvec=CAP)
    if c["precision"] == "mixed":
        o["inner_tol"] = 1e-5 if c["kind"] == "sweep" else 1e-4
    if c["kind"] == "schwarz":
        o = dict(method="schwarz", restart=100, tol=1e-10, max_matvec=2000, inner_tol=1e-13, inner_restart=4,
                 dd_inner=c["method"])
    return o


def prepare(c, seed):
    mesh, beta, g, eta, rec, x = _inputs(c, seed)
    how = {} if c["mesh"] == "box" else dict(order="rcm", sigma=256)
    if c["kind"] == "schwarz":
        how["parts"] = (2, 2, 1)
    model = Helmholtz(mesh, beta, eta=eta, gls=c["gls"], dirichlet=c["dirichlet"], **how)
    dev = lambda a: torch.as_tensor(a, device="cuda")  # noqa: E731
    s = dict(kind=c["kind"], model=model, g=dev(g), freqs=_freqs(c), opts=_opts(c))
    if c["kind"] == "product":
        model.set_frequency(c["freq"])
        s["x"] = dev(x)
    elif c["kind"] == "sweep":
        s["F"] = model.load(s["g"])[:, None].expand(-1, c["nfreq"]).contiguous()
    elif c["kind"] == "gradient":
        s["beta"] = dev(np.stack([beta.real, beta.imag], 1)).requires_grad_()
        s["eta"] = dev(eta).requires_grad_()
        s["rec"] = dev(rec)
    return s


def run(s):
    model, kind = s["model"], s["kind"]
    if kind == "product":
        return model.apply(s["x"])
    if kind == "sweep":
        P, _ = model.solve_sweep(s["freqs"], s["F"], **s["opts"])
        return P
    if kind == "gradient":
        J = HelmholtzEnergy.apply(s["beta"], s["eta"], model, s["freqs"], s["g"], s["rec"], s["opts"])
        db, de = torch.autograd.grad(J, (s["beta"], s["eta"]))
        return {"J": J.detach(), "dbeta": db, "deta": de}
    model.set_frequency(s["freqs"][0])
    p, _ = model.solve(model.load(s["g"]), **s["opts"])
    return p


# ---------------------------------------------------------------- the same in plain torch
def _element_matrices(X):
    """(K, M) per element: X [e, 8, 3] trilinear hexahedra (2 x 2 x 2 Gauss) or [e, 4, 3] linear tetrahedra."""
    if X.shape[1] == 4:
        D = (X[:, 1:] - X[:, :1]).transpose(1, 2)
        vol = torch.linalg.det(D).abs() / 6.0
        G = torch.linalg.inv(D)
        G = torch.cat([-G.sum(1, keepdim=True), G], 1)
        M = (torch.ones(4, 4, dtype=X.dtype, device=X.device) + torch.eye(4, dtype=X.dtype, device=X.device)) / 20.0
        return vol[:, None, None] * torch.matmul(G, G.transpose(1, 2)), vol[:, None, None] * M
    K = torch.zeros(X.shape[0], 8, 8, dtype=X.dtype, device=X.device)
    M = torch.zeros_like(K)
    corner = [[2 * ((a >> d) & 1) - 1 for d in range(3)] for a in range(8)]
    q = 1.0 / math.sqrt(3.0)
    for sx, sy, sz in corner:
        r = (sx * q, sy * q, sz * q)
        N, dN = [], []
        for c in corner:
            t = [1.0 + r[d] * c[d] for d in range(3)]
            N.append(t[0] * t[1] * t[2] / 8.0)
            dN.append([c[0] * t[1] * t[2] / 8.0, t[0] * c[1] * t[2] / 8.0, t[0] * t[1] * c[2] / 8.0])
        N = torch.tensor(N, dtype=X.dtype, device=X.device)
        J = torch.matmul(torch.tensor(dN, dtype=X.dtype, device=X.device).T, X)
        det = torch.linalg.det(J).abs()[:, None, None]
        B = torch.linalg.solve(J, torch.tensor(dN, dtype=X.dtype, device=X.device).T.expand(X.shape[0], 3, 8))
        K += det * torch.matmul(B.transpose(1, 2), B)
        M += det * torch.outer(N, N)
    return K, M


def _face_mass(X):
    """Mass matrix per boundary face: plane quadrilaterals [f, 4, 3] in tensor order, or triangles [f, 3, 3]."""
    e = dict(dtype=X.dtype, device=X.device)
    if X.shape[1] == 3:
        area = torch.linalg.cross(X[:, 1] - X[:, 0], X[:, 2] - X[:, 0]).norm(dim=1) / 2.0
        return area[:, None, None] * (torch.ones(3, 3, **e) + torch.eye(3, **e)) / 12.0
    out = torch.zeros(X.shape[0], 4, 4, **e)
    q = 1.0 / math.sqrt(3.0)
    for u in (-q, q):
        for v in (-q, q):
            s = [(2 * (a & 1) - 1, 2 * (a >> 1) - 1) for a in range(4)]
            N = torch.tensor([(1 + u * a) * (1 + v * b) / 4 for a, b in s], **e)
            du = torch.tensor([a * (1 + v * b) / 4 for a, b in s], **e)
            dv = torch.tensor([b * (1 + u * a) / 4 for a, b in s], **e)
            J = torch.linalg.cross((du[:, None] * X).sum(1), (dv[:, None] * X).sum(1)).norm(dim=1)
            out += J[:, None, None] * torch.outer(N, N)
    return out


class _Plain:
    """The discrete problem in FP64, element by element."""

    def __init__(self, c, seed):
        mesh, beta, g, eta, rec, x = _inputs(c, seed)
        dev = lambda a, t=None: torch.as_tensor(np.ascontiguousarray(a), dtype=t, device="cuda")  # noqa: E731
        self.c, self.beta, self.n = c, beta, mesh["n_nodes"]
        self.elems = dev(mesh.get("tet", mesh.get("hex")), torch.int64)
        X = dev(mesh["xyz"])
        self.K, self.M = _element_matrices(X[self.elems])
        self.faces, self.tag = dev(mesh["bface"], torch.int64), dev(mesh["bface_tag"], torch.int64)
        self.src = dev(mesh["bface_src"].astype(np.int64)) == 1
        self.F = _face_mass(X[self.faces])
        self.g, self.rec = dev(g), dev(rec)
        self.eta = None if eta is None else dev(eta)
        self.x = None if x is None else dev(x)
        self.h = mesh["h"]
        self.dir = torch.zeros(self.n, dtype=torch.bool, device="cuda")
        if c["dirichlet"]:
            self.dir[self.faces[self.src].reshape(-1)] = True
        npe = self.elems.shape[1]
        pairs = [(a, b) for b in range(npe) for a in range(b)] if npe == 4 else \
            [(a, a | (1 << d)) for a in range(8) for d in range(3) if not a & (1 << d)]
        E = X[self.elems]
        self.edge = float(torch.stack([(E[:, a] - E[:, b]).norm(dim=1) for a, b in pairs]).mean())

    def mass(self, k):
        if not self.c["gls"]:
            return k * k
        t = k * self.edge
        return k * k * 6.0 * (1.0 - math.cos(t)) / (t * t * (2.0 + math.cos(t)))

    def wall(self, k):
        return 1j * k * torch.as_tensor(self.beta, device="cuda")[self.tag]

    @staticmethod
    def _add(y, nodes, mats, x, scale=None):
        v = x[nodes]
        v = torch.complex((mats * v.real[:, None, :]).sum(2), (mats * v.imag[:, None, :]).sum(2))
        if scale is not None:
            v = scale[:, None] * v
        y.index_add_(0, nodes.reshape(-1), v.reshape(-1))

    def raw(self, k, x):
        y = torch.zeros_like(x)
        m = self.mass(k)
        for at in range(0, self.elems.shape[0], 1 << 18):
            e = slice(at, at + (1 << 18))
            self._add(y, self.elems[e], self.K[e] - m * self.M[e], x)
            if self.eta is not None:
                self._add(y, self.elems[e], self.M[e], x, 1j * k * k * self.eta[e])
        self._add(y, self.faces, self.F, x, self.wall(k))
        return y

    def apply(self, k, x):
        if not self.c["dirichlet"]:
            return self.raw(k, x)
        y = self.raw(k, torch.where(self.dir, 0.0, x))
        return torch.where(self.dir, x, y)

    def load(self, k):
        if self.c["dirichlet"]:
            gd = torch.where(self.dir, self.g, 0.0)
            return torch.where(self.dir, gd, -self.raw(k, gd))
        f = torch.zeros_like(self.g)
        self._add(f, self.faces[self.src], self.F[self.src], self.g)
        return f

    def solve(self, k, f):
        P = self._separable(k) if self.c["mesh"] == "box" and not self.c["dirichlet"] else self._dense(k)
        A = lambda v: self.apply(k, v)  # noqa: E731
        x = P(f)
        for _ in range(3):
            x = x + _gmres(A, P, f - A(x))
        return x

    def _dense(self, k):
        n = self.n
        A = torch.zeros(n * n, dtype=torch.complex128, device="cuda")
        m = self.mass(k)

        def put(nodes, mats):
            A.index_add_(0, (nodes[:, :, None] * n + nodes[:, None, :]).reshape(-1), mats.reshape(-1))

        put(self.elems, (self.K - m * self.M).to(torch.complex128))
        if self.eta is not None:
            put(self.elems, 1j * k * k * self.eta[:, None, None] * self.M)
        put(self.faces, self.wall(k)[:, None, None] * self.F)
        A = A.reshape(n, n)
        A[self.dir, :] = 0.0
        A[:, self.dir] = 0.0
        A[self.dir, self.dir] = 1.0
        lu = torch.linalg.lu_factor(A)
        return lambda f: torch.linalg.lu_solve(*lu, f[:, None])[:, 0]

    def _separable(self, k):
        """A^-1 of the box without an absorption field, from the eigenvectors of its three one-dimensional problems."""
        V, lam = [], []
        for d, ne in enumerate((self.c["nx"], self.c["ny"], self.c["nz"])):
            h = self.h[d]
            i = np.arange(ne)
            K, M = np.zeros((ne + 1, ne + 1)), np.zeros((ne + 1, ne + 1))
            for a in range(2):
                for b in range(2):
                    np.add.at(K, (i + a, i + b), (1.0 if a == b else -1.0) / h)
                    np.add.at(M, (i + a, i + b), h / (3.0 if a == b else 6.0))
            K = K.astype(np.complex128)
            K[0, 0] += 1j * k * self.beta[2 * d]
            K[-1, -1] += 1j * k * self.beta[2 * d + 1]
            L = np.linalg.cholesky(M)
            Li = np.linalg.inv(L)
            w, U = np.linalg.eig(Li @ K @ Li.T)
            U = U / np.sqrt((U * U).sum(0))
            V.append(torch.as_tensor(Li.T @ U, device="cuda"))
            lam.append(torch.as_tensor(w, device="cuda"))
        D = lam[2][:, None, None] + lam[1][None, :, None] + lam[0][None, None, :] - self.mass(k)

        def along(Z, mats):
            Z = torch.matmul(Z, mats[0])
            Z = torch.matmul(Z.transpose(1, 2), mats[1]).transpose(1, 2)
            return torch.matmul(Z.permute(1, 2, 0), mats[2]).permute(2, 0, 1)

        def inverse(f):
            Z = along(f.reshape(D.shape), V) / D
            return along(Z, [v.T for v in V]).reshape(-1).contiguous()

        return inverse


def _gmres(A, P, r, m=40):
    """Right-preconditioned GMRES(m) correction for the residual r."""
    beta = float(r.norm())
    if beta == 0.0:
        return torch.zeros_like(r)
    Q, Z, H = [r / beta], [], np.zeros((m + 1, m), dtype=np.complex128)
    for j in range(m):
        Z.append(P(Q[j]))
        w = A(Z[j])
        for _ in range(2):
            for i, q in enumerate(Q):
                t = complex(torch.vdot(q, w))
                H[i, j] += t
                w = w - t * q
        H[j + 1, j] = float(w.norm())
        e = np.zeros(j + 2, dtype=np.complex128)
        e[0] = beta
        y = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
        if np.linalg.norm(e - H[:j + 2, :j + 1] @ y) < 1e-13 * beta or abs(H[j + 1, j]) < 1e-14 * beta:
            break
        Q.append(w / float(H[j + 1, j].real))
    return sum(complex(t) * z for t, z in zip(y, Z))


def exact(c, seed):
    # without the box's eigenvectors only a small system is solved directly
    if c["kind"] != "product" and (c["mesh"] != "box" or c["dirichlet"]) and _counts(c)[0] > DENSE:
        return None
    p = _Plain(c, seed)
    ks = [float(W.wavenumber(f)) for f in _freqs(c)]
    if c["kind"] == "product":
        return p.apply(ks[0], p.x)
    if c["kind"] == "sweep":
        return torch.stack([p.solve(k, p.load(k)) for k in ks], 1)
    if c["kind"] != "gradient":
        return p.solve(ks[0], p.load(ks[0]))
    J, db = 0.0, np.zeros((6, 2))
    de = torch.zeros(p.elems.shape[0], dtype=torch.float64, device="cuda")
    for k in ks:
        u = p.solve(k, p.load(k))
        gr = torch.zeros_like(u)
        gr[p.rec] = u[p.rec]
        J += float((u[p.rec].abs() ** 2).sum())
        lam = p.solve(k, gr.conj().resolve_conj()).conj().resolve_conj()
        ue, le = u[p.elems], lam[p.elems]
        de += 2 * k * k * (le.conj() * torch.matmul(p.M.to(ue.dtype), ue[:, :, None])[:, :, 0]).sum(1).imag
        uf, lf = u[p.faces], lam[p.faces]
        t = (lf.conj() * torch.matmul(p.F.to(uf.dtype), uf[:, :, None])[:, :, 0]).sum(1)
        for w in range(6):
            s = complex(t[p.tag == w].sum())
            db[w] += [2 * k * s.imag, 2 * k * s.real]
    return {"J": torch.tensor(J, dtype=torch.float64, device="cuda"), "dbeta": torch.as_tensor(db), "deta": de}
