"""Scalar steps by kernels of their own (large systems, more than 1,024 blocks
of 256 rows): solves that converge, stop at the product cap, and run on past
rounding level through breakdowns and restarts, in the stored forms.  The
residual is recomputed with another context's product, the tensor form's."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZE = (67, 62, 61)      # 265,608 nodes: 1,038 blocks
METHODS = [("bicgstab", {}), ("bicgstabl", dict(restart=1)), ("bicgstabl", dict(restart=5)), ("tfqmr", {}),
           ("tfqmr", dict(precision="mixed", inner_tol=1e-3))]


@pytest.fixture(scope="module")
def systems():
    import paper_2112_00087_amd as P
    mesh = W.box_mesh(*SIZE)
    beta = 0.03 * np.ones(6)
    mp = pytest.MonkeyPatch()
    out = {}
    for form, on in (("tensor", "1"), ("stored", "0")):
        mp.setenv("HZ_TENSOR", on)
        out[form] = P.Helmholtz(mesh, beta)
        out[form].set_frequency(45.0)
    mp.undo()
    g = np.zeros(mesh["n_nodes"], np.complex128)
    pn = W.patch_nodes(mesh)
    g[pn] = np.random.default_rng(1).standard_normal(pn.size)
    out["f"] = out["tensor"].load(torch.as_tensor(g, device="cuda"))
    yield out
    for form in ("tensor", "stored"):
        out[form].close()


@pytest.mark.parametrize("method,kw", METHODS)
def test_large_stored_solves(systems, method, kw):
    m, other, f = systems["stored"], systems["tensor"], systems["f"]
    for what, opts in (("converged", dict(tol=1e-6, max_matvec=20000)), ("capped", dict(tol=1e-6, max_matvec=61)),
                       ("past rounding", dict(tol=1e-30, max_matvec=2500))):
        print("large stored", method, kw, what, flush=True)
        p, info = m.solve(f, method=method, **kw, **opts)
        rel = float((f - other.apply(p)).norm() / f.norm())
        print("  ", info, rel, flush=True)
        assert abs(info["relres_true"] - rel) <= 1e-3 * rel + 1e-13
        assert info["status"] == (0 if what == "converged" else 1)
        assert rel <= (1e-6 if what == "converged" else 1.0 if what == "capped" else 1e-10)
