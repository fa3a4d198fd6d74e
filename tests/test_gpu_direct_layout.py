"""Operators on small lattices read and write the caller's layout directly; vectors that are not 16-byte
aligned (and larger lattices) go through conversion passes.  Both routes give the same bits."""
import math

import pytest
import torch

from gpu_util import Case, flush, need_gpu

pytestmark = pytest.mark.gpu


def vectors(n, dtype, off):
    """Input and output of n reals starting `off` reals after a 16-byte boundary."""
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.float64).to(dtype)
    buf, out = (torch.zeros(n + 4, device="cuda", dtype=dtype) for _ in range(2))
    buf[off:off + n] = x
    return buf[off:off + n], out[off:off + n]


@pytest.mark.parametrize("dims,cstar,block", [((4, 4, 4, 4), 0, (2, 4, 2, 2)), ((6, 6, 6, 10), 0, (3, 2, 6, 10)),
                                              ((4, 8, 6, 12), 2, (4, 4, 3, 4))], ids=str)
def test_direct_layout_bitwise_the_converted(dims, cstar, block):
    need_gpu()
    flush(f"[gpu] direct layout {dims} cstar {cstar}")
    c = Case(dims, seed=23, bc_phase=(math.pi, 0.1, -0.3, 0.2), cstar=cstar)
    c.D.set_cache_block(block)
    for prec, dtype, off in (("f64", torch.float64, 1), ("f32", torch.float32, 2)):
        for dagger in (False, True):
            for layout in ("lex", "eo", "openqxd"):
                (x, y), (xo, yo) = vectors(c.V * 24, dtype, 0), vectors(c.V * 24, dtype, off)
                c.D.apply(y, x, prec, layout, dagger)
                c.D.apply(yo, xo, prec, layout, dagger)
                assert torch.equal(y, yo) and float(y.abs().max()) > 0, (prec, dagger, layout)
                if layout == "lex":
                    continue
                (x, y), (xo, yo) = vectors(c.V * 12, dtype, 0), vectors(c.V * 12, dtype, off)
                c.D.apply_eo(y, x, prec, layout, dagger)
                c.D.apply_eo(yo, xo, prec, layout, dagger)
                assert torch.equal(y, yo) and float(y.abs().max()) > 0, (prec, dagger, layout)
    c.D.close()
