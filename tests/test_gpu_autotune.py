"""A product variant that was forced is not what later sweeps run: neither in
the same context nor, through the cache file, in another."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TENSOR = 20000000        # variant codes of the tensor form start here


def test_forced_variants_are_not_kept(monkeypatch, tmp_path):
    import paper_2112_00087_amd as P
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("HZ_AUTOTUNE_CACHE", str(cache))
    mesh = W.box_mesh(12, 9, 8)
    freqs = np.linspace(50.0, 120.0, 5)
    X = torch.randn(mesh["n_nodes"], freqs.size, dtype=torch.complex128, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(3))
    m = P.Helmholtz(mesh, 0.02 * np.ones(6))
    for staged in ("1", "0"):
        monkeypatch.setenv("HZ_SPMM_STAGED", staged)
        Y, code = m.apply_sweep(freqs, X)
        assert code < TENSOR
        assert not cache.exists() or cache.read_text() == ""
    monkeypatch.delenv("HZ_SPMM_STAGED")
    Z, own = m.apply_sweep(freqs, X)
    assert own > TENSOR and float((Y - Z).norm() / Z.norm()) < 1e-13
    m.close()
    # a file that holds such an entry for this shape
    line = cache.read_text().splitlines()[-1]
    cache.write_text(f"{line.rpartition('|')[0]}|{code}\n")
    m = P.Helmholtz(mesh, 0.02 * np.ones(6))
    assert m.apply_sweep(freqs, X)[1] > TENSOR
    m.close()
