"""Calls on small lattices that read the caller's layout directly leave behind what the same call on other vectors
needs under graph capture, where nothing may be allocated."""
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
