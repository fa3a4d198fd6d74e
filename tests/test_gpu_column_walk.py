"""The column walk on lattices whose time extent is no multiple of the chunk length and whose spatial blocks
do not divide among the eight XCDs: bitwise the single applies."""
import pytest
import torch

from gpu_util import Case, flush, need_gpu

pytestmark = pytest.mark.gpu


# 6 and 9 spatial blocks (two XCDs without one, or one with two and the rest with one); 10 and 14 time slices in
# chunks of at least three, the last one shorter; 2 slices: one chunk
@pytest.mark.parametrize("dims", [(10, 6, 8, 16), (14, 6, 12, 16), (2, 6, 12, 16)], ids=lambda d: "x".join(map(str, d)))
def test_column_walk_uneven(monkeypatch, dims):
    need_gpu()
    flush(f"[gpu] column walk {dims}")
    c = Case(dims, seed=31)
    for prec in ("f32", "bf16"):
        n = c.D.native_empty(prec, 1).numel()
        g = torch.Generator(device="cuda").manual_seed(1)
        x = torch.randn(12 * n, generator=g, device="cuda").to(c.D.native_empty(prec, 1).dtype)
        monkeypatch.setenv("DIRAC_HOP_SHAPE", "5")
        want = torch.zeros_like(x)
        for r in range(12):
            c.D.apply_eo(want[r * n:(r + 1) * n], x[r * n:(r + 1) * n], prec, "native")
        for shape in range(41, 48):
            monkeypatch.setenv("DIRAC_HOP_SHAPE", str(shape))
            for nr in (12, 5):
                out = torch.zeros_like(x)
                c.D.apply_eo_multi(out[:nr * n], x[:nr * n], nr, prec)
                assert torch.equal(out[:nr * n], want[:nr * n]), (prec, shape, nr)
    c.D.close()
