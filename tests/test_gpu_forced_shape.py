"""A launch shape forced by DIRAC_HOP_SHAPE is taken on small lattices and user layouts too."""
import pytest
import torch

from gpu_util import Case, flush, need_gpu
from test_gpu_direct_layout import vectors

pytestmark = pytest.mark.gpu


def test_forced_shape_is_taken(monkeypatch):
    need_gpu()
    flush("[gpu] forced shape on a small lattice")
    c = Case((4, 4, 6, 8), seed=24)
    x, y = vectors(c.V * 12, torch.float64, 0)
    z = torch.zeros_like(y)

    def kernels(out):
        c.D.apply_eo(out, x, "f64", "eo")
        torch.cuda.synchronize()
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
            c.D.apply_eo(out, x, "f64", "eo")
            torch.cuda.synchronize()
        return [e.key for e in prof.key_averages()]

    assert any("k_hop_d" in k for k in kernels(y))
    monkeypatch.setenv("DIRAC_HOP_SHAPE", "8")
    names = kernels(z)
    assert any("k_hop" in k for k in names) and not any("k_hop_d" in k for k in names), names
    assert torch.equal(y, z)
    c.D.close()
