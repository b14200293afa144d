"""Solver iterations replayed as HIP graphs give the bits of the launches.

One context with graphs, one without (HZ_GRAPH=0).  Solves alternate over
right-hand sides, frequencies, methods and parameters, so captures are
replayed, replaced and replayed again, with eager work and synchronisations of
the caller's between them."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

METHODS = [("gmres", dict(restart=8)), ("bicgstab", {}), ("bicgstabl", dict(restart=4)), ("tfqmr", {}),
           ("tfqmr", dict(precision="mixed", inner_tol=1e-3))]


@pytest.mark.parametrize("form", ["tensor", "stored"])
@pytest.mark.parametrize("method,kw", METHODS)
def test_replays_match_launches(monkeypatch, form, method, kw):
    import paper_2112_00087_amd as P
    print("replay", form, method, kw, flush=True)
    monkeypatch.setenv("HZ_TENSOR", "1" if form == "tensor" else "0")
    rng = np.random.default_rng(4)
    mesh = W.box_mesh(12, 9, 8)
    beta = rng.uniform(0.01, 0.05, 6) + 0.01j
    ctx = []
    for on in ("1", "0"):
        monkeypatch.setenv("HZ_GRAPH", on)
        ctx.append(P.Helmholtz(mesh, beta))
    n = mesh["n_nodes"]
    opts = dict(method=method, tol=1e-9, max_matvec=400, **kw)
    scratch = torch.zeros(1 << 20, device="cuda")
    for step in range(6):
        f = torch.as_tensor(rng.standard_normal(n) + 1j * rng.standard_normal(n), device="cuda")
        if step == 3:
            for m in ctx:
                m.set_params(2.0 * beta, None)
        out = []
        for m in ctx:
            m.set_frequency(70.0 + 15.0 * (step % 2))
            out.append(m.solve(f, **opts))
            scratch.add_(1.0).sum().item()
            if step == 2:   # another capture under another tag in between
                m.solve(f, method="bicgstab" if method != "bicgstab" else "tfqmr", tol=1e-6, max_matvec=200)
        (p, a), (q, b) = out
        assert a["status"] == b["status"] and a["matvecs"] == b["matvecs"]
        assert torch.equal(torch.view_as_real(p), torch.view_as_real(q))
    for m in ctx:
        m.close()
