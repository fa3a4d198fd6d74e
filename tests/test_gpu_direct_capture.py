"""Calls on small lattices that read the caller's layout directly leave behind what the same call on other vectors
needs under graph capture, where nothing may be allocated, and a forced launch shape is still taken."""
import pytest
import torch

from gpu_util import Case, flush, need_gpu
from test_gpu_direct_layout import vectors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["apply", "apply_eo"])
def test_unaligned_call_captured_after_aligned_one(op):
    need_gpu()
    flush(f"[gpu] captured unaligned {op}")
    c = Case((4, 4, 6, 8), seed=24)
    n = c.V * 24 if op == "apply" else c.V * 12
    f = getattr(c.D, op)
    (x, y), (xo, yo) = vectors(n, torch.float32, 0), vectors(n, torch.float32, 2)
    f(y, x, "f32", "eo")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        f(yo, xo, "f32", "eo")
    for k in range(3):
        xo.copy_(x * (k + 1))
        yo.zero_()
        graph.replay()
        torch.cuda.synchronize()
        f(y, x * (k + 1), "f32", "eo")
        assert torch.equal(y, yo) and float(y.abs().max()) > 0
    c.D.close()


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
