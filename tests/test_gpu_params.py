"""A set_params call that is refused leaves the context as it was: the formed
operator, the operator formed again at the same and at another frequency, and
the sweep's, in the tensor and in the stored forms."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("form", ["tensor", "stored", "reordered"])
@pytest.mark.parametrize("first_eta", [False, True])
@pytest.mark.parametrize("bad", ["eta", "beta"])
def test_refused_parameters_change_nothing(monkeypatch, form, first_eta, bad):
    import paper_2112_00087_amd as P
    print("refused parameters", form, first_eta, bad, flush=True)
    if form == "stored":
        monkeypatch.setenv("HZ_TENSOR", "0")
    how = dict(order="rcm") if form == "reordered" else {}
    rng = np.random.default_rng(8)
    mesh = W.box_mesh(11, 8, 7)
    beta, other = rng.uniform(0.01, 0.05, (2, 6)) + 1j * rng.uniform(-0.01, 0.01, (2, 6))
    e0, e1 = rng.uniform(0.0, 0.02, (2, mesh["n_elems"]))
    m, fresh = (P.Helmholtz(mesh, beta, eta=e0 if first_eta else None, **how) for _ in range(2))
    for q in (m, fresh):
        q.set_frequency(110.0)
    x = torch.as_tensor(rng.standard_normal(m.n) + 1j * rng.standard_normal(m.n), device="cuda")
    X = x[:, None].expand(-1, 3).contiguous()
    freqs = [50.0, 100.0, 150.0]
    m.apply_sweep(freqs, X)          # a sweep built before the refused call
    if bad == "eta":
        e1[-1] = np.nan
    else:
        other[5] = np.inf
    m.set_frequency(110.0)
    with pytest.raises(P.HzError):
        m.set_params(other, e1)
    same = lambda a, b: torch.equal(torch.view_as_real(a), torch.view_as_real(b))  # noqa: E731
    assert same(m.apply(x), fresh.apply(x))          # the operator formed before still stands
    for f in (110.0, 140.0):
        for q in (m, fresh):
            q.set_frequency(f)
        assert same(m.apply(x), fresh.apply(x))
        assert same(m.diag(), fresh.diag())
    # (two contexts may tune different product variants: other summation orders)
    a, b = (q.apply_sweep(freqs, X)[0] for q in (m, fresh))
    assert float((a - b).norm() / b.norm()) < 1e-14
    # accepted parameters reach all of them
    e1[-1], other[5] = 0.01, 0.02
    m.set_params(other, e1)
    new = P.Helmholtz(mesh, other, eta=e1, **how)
    for q in (m, new):
        q.set_frequency(110.0)
    assert same(m.apply(x), new.apply(x))
    a, b = (q.apply_sweep(freqs, X)[0] for q in (m, new))
    assert float((a - b).norm() / b.norm()) < 1e-14
    for q in (m, fresh, new):
        q.close()
