"""When solver iterations are captured as HIP graphs and when a kept capture is
replayed: one capture serves a loop over frequencies and parameters,
and none is made before the same run has come up a few times.  (That replays
give the launches' bits: test_gpu_replay.py; here also for captures kept from an
earlier solve.)"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

METHODS = [("gmres", dict(restart=8)), ("bicgstab", {}), ("bicgstabl", dict(restart=4)), ("tfqmr", {})]


def _pair(monkeypatch, mesh, beta, eta):
    """A context with graphs and one without."""
    import paper_2112_00087_amd as P
    out = []
    for on in ("1", "0"):
        monkeypatch.setenv("HZ_GRAPH", on)
        out.append(P.Helmholtz(mesh, beta, eta=eta))
    return out


@pytest.mark.parametrize("form", ["tensor", "absorption", "stored"])
@pytest.mark.parametrize("method,kw", METHODS)
def test_one_capture_serves_all_frequencies(monkeypatch, form, method, kw):
    print("replay counts", form, method, flush=True)
    monkeypatch.setenv("HZ_TENSOR", "0" if form == "stored" else "1")
    rng = np.random.default_rng(6)
    mesh = W.box_mesh(12, 9, 8)
    beta = rng.uniform(0.01, 0.05, 6) + 0.01j
    eta = rng.uniform(0.0, 0.02, mesh["n_elems"]) if form == "absorption" else None
    on, off = _pair(monkeypatch, mesh, beta, eta)
    scratch = torch.zeros(1 << 20, device="cuda")
    last = 0
    for step, freq in enumerate((70.0, 85.0, 85.0, 100.0, 115.0)):
        if step == 2:      # new parameters at the same frequency: the kept capture, new tables
            for m in (on, off):
                m.set_params(2.0 * beta, None if eta is None else 0.5 * eta)
        f = torch.as_tensor(rng.standard_normal(on.n) + 1j * rng.standard_normal(on.n), device="cuda")
        got = []
        for m in (on, off):
            m.set_frequency(freq)
            got.append(m.solve(f, method=method, tol=1e-30, max_matvec=400, **kw))
            scratch.add_(1.0).sum().item()
        (p, a), (q, b) = got
        assert a["matvecs"] == b["matvecs"]
        assert torch.equal(torch.view_as_real(p), torch.view_as_real(q))
        captures, replays = on.replay_counts()
        assert captures == 1 and replays > last, (step, captures, replays)
        last = replays
    assert off.replay_counts() == (0, 0)
    for m in (on, off):
        m.close()


@pytest.mark.parametrize("method,kw", METHODS)
def test_short_solves_capture_on_repetition(monkeypatch, method, kw):
    """Two full chunks (five BiCGStab(4) cycles, one GMRES cycle) a solve: the first
    solve captures nothing, a few alike make one capture."""
    rng = np.random.default_rng(7)
    mesh = W.box_mesh(12, 9, 8)
    on, off = _pair(monkeypatch, mesh, 0.02 * np.ones(6), None)
    f = torch.as_tensor(rng.standard_normal(on.n) + 0j, device="cuda")
    for step, freq in enumerate((70.0, 85.0, 100.0) * 3):
        on.set_frequency(freq)
        on.solve(f, method=method, tol=1e-30, max_matvec={"gmres": 9, "bicgstabl": 48}.get(method, 72), **kw)
        captures, replays = on.replay_counts()
        if step == 0:
            assert (captures, replays) == (0, 0)
    assert captures == 1 and replays >= 1
    for m in (on, off):
        m.close()
