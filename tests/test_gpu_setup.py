"""Contexts made from the memory of earlier ones: fields of a context do not depend on what its
memory held before, and two live contexts never share memory."""
import pytest
import torch

from gpu_util import Case, flush, need_gpu

pytestmark = pytest.mark.gpu


def fields(c, prec):
    x = c.D.native_empty(prec, 1)
    x.copy_(torch.linspace(-1.0, 1.0, x.numel(), dtype=torch.float64, device="cuda").to(x.dtype))
    y = torch.zeros_like(x)
    c.D.apply_eo(y, x, prec, "native")
    used = c.D.vh // 64 * 64 * 24  # whole site blocks: padding sites are not written
    return [c.D.clover(), c.D.clover(inverse=True), y[:used].clone()]


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (6, 6, 6, 10)], ids=lambda d: "x".join(map(str, d)))
def test_contexts_reuse_memory(dims):
    need_gpu()
    flush(f"[gpu] context memory {dims}")
    want = {}
    for seed in (11, 12):  # two gauge fields, each alone
        c = Case(dims, seed=seed)
        want[seed] = [fields(c, p) for p in ("f64", "f32", "bf16")]
        c.D.close()
    a, b = Case(dims, seed=12), Case(dims, seed=11)  # both alive, in the memory of the two before
    for c, seed in ((a, 12), (b, 11), (a, 12)):
        got = [fields(c, p) for p in ("f64", "f32", "bf16")]
        for w, g in zip(want[seed], got):
            assert all(torch.equal(x, y) for x, y in zip(w, g)), seed
    a.D.close()
    b.D.close()
