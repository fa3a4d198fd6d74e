"""Conversions between the caller's site order and the planes: blocks of 64 sites, both parities in one pass.
FP64 fields come back bit for bit; vectors that start at any real give the bits of aligned ones."""
import math

import pytest
import torch

from gpu_util import Case, flush, need_gpu

pytestmark = pytest.mark.gpu


# Sites per parity: 8 (one partial block), 64 (one full), 1080 (remainder 56), 18,144 (above the direct path, remainder 32).
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 4, 4, 4), (6, 6, 10, 6), (18, 14, 12, 12)], ids=str)
def test_fields_come_back(dims):
    need_gpu()
    flush(f"[gpu] site layouts {dims}")
    c = Case(dims, seed=31, bc_phase=(math.pi, 0.1, -0.3, 0.2))
    c.D.set_cache_block(tuple(d // 2 if d > 4 and m < 3 else d for m, d in enumerate(dims)))
    g = torch.Generator(device="cuda").manual_seed(5)
    for layout in ("lex", "eo", "openqxd"):
        f = torch.randn(c.V * 72, generator=g, device="cuda", dtype=torch.float64)
        c.D.load_clover(f, layout)
        assert torch.equal(c.D.clover(layout=layout).reshape(-1), f), layout
        for prec, dtype in (("f64", torch.float64), ("f32", torch.float32)):
            x = torch.randn(c.V * 24 + 4, generator=g, device="cuda", dtype=torch.float64).to(dtype)
            y, yo = torch.zeros_like(x), torch.zeros_like(x)
            a = x[:c.V * 24]
            xo = torch.empty_like(x)
            xo[1:1 + a.numel()] = a
            c.D.apply(y[:a.numel()], a, prec, layout)
            c.D.apply(yo[1:1 + a.numel()], xo[1:1 + a.numel()], prec, layout)
            assert torch.equal(y[:a.numel()], yo[1:1 + a.numel()]) and float(y.abs().max()) > 0, (prec, layout)
            assert float(y[a.numel():].abs().max()) == 0 and float(yo[0]) == 0, (prec, layout)
    c.D.close()
