"""A gauge field that starts 8 bytes after a 16-byte boundary (a view into a larger allocation), and angles that start
4 bytes after an 8-byte one, give the context of aligned ones, bit for bit."""
import math

import pytest
import torch

import gen
import paper_2502_02490_amd as P
from gpu_util import flush, need_gpu, to_dev

pytestmark = pytest.mark.gpu


def shifted(t, off):
    """The bytes of t as a contiguous tensor that starts `off` bytes after a 16-byte boundary."""
    raw = t.contiguous().view(torch.float32).reshape(-1) if t.dtype == torch.float64 else torch.view_as_real(t).view(torch.float32).reshape(-1)
    buf = torch.zeros(raw.numel() + 8, dtype=torch.float32, device="cuda")
    buf[off // 4:off // 4 + raw.numel()] = raw
    out = buf[off // 4:off // 4 + raw.numel()]
    assert out.data_ptr() % 16 == off
    return out


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 6, 6, 10)], ids=lambda d: "x".join(map(str, d)))
def test_unaligned_gauge_field(dims):
    need_gpu()
    flush(f"[gpu] unaligned links {dims}")
    U, th = to_dev(gen.su3_field(dims, 0.4, 5)), to_dev(gen.u1_field(dims, 0.3, 5))
    b = to_dev(gen.gaussian_spinor(dims, 6))
    got = []
    for u, a in ((U, th), (shifted(U, 8), shifted(th, 8)), (shifted(U, 4), shifted(th, 4))):
        with P.Dirac(u, a, dims, 0.12, 1.2, 1.0, -1, (math.pi, 0.1, 0.0, 0.0)) as D:
            y = torch.zeros_like(b)
            D.apply(y, b, "f64", "lex")
            got.append((D.clover(), D.clover(inverse=True), y))
    for g in got[1:]:
        assert all(torch.equal(p, q) for p, q in zip(got[0], g))
