"""The GCR step at the edges of its launch rules, and on Krylov spaces that end before the cycle does."""
import math

import numpy as np
import pytest
import torch

import gen
import paper_2502_02490_amd as P
from gpu_util import flush, need_gpu, to_dev

pytestmark = pytest.mark.gpu


# 128 sites per parity (two chunks); 1080 (a ragged last chunk); 32,768 and 36,864 (64-site chunks over eight
# wavefronts up to 32,768); 131,072 (work-groups of 512)
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 6, 6, 10), (16, 16, 16, 16), (18, 16, 16, 16), (32, 32, 16, 16)],
                         ids=lambda d: "x".join(map(str, d)))
def test_solutions_at_launch_edges(dims):
    """Each solve's residual, recomputed by the FP64 operator, is below the tolerance it was asked for; restarts
    of 1, 9 and 40 exercise no, one and several basis vectors per wavefront."""
    need_gpu()
    flush(f"[gpu] GCR step {dims}")
    U, th = gen.su3_field(dims, 0.4, 5), gen.u1_field(dims, 0.3, 5)
    b = to_dev(gen.gaussian_spinor(dims, 6))
    with P.Dirac(to_dev(U), to_dev(th), dims, 0.12, 1.2, 1.0, -1) as D:
        bn, xn, rn = (D.native_empty("f64") for _ in range(3))
        D.to_native(b, "f64", "lex", out=bn)
        for kw in (dict(method=P.GCR, restart=1), dict(method=P.GCR, restart=9), dict(method=P.GCR, restart=40),
                   dict(method=P.MIXED_GCR, inner_prec="f32", restart=9),
                   dict(method=P.MIXED_GCR, inner_prec="f16", restart=12),
                   dict(method=P.MIXED_GCR, inner_prec="bf16", restart=40)):
            x = torch.zeros_like(b)
            info = D.solve(x, b, tol=1e-11, **kw)
            D.to_native(x, "f64", "lex", out=xn)
            assert D.residual(rn, bn, xn, rel=True) < 1e-11 and info.fell_back == 0, (kw, info.true_rel_res)


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 16, 18)], ids=lambda d: "x".join(map(str, d)))
def test_krylov_space_exhausted(dims):
    """Unit links and periodic boundaries: a sum of two plane waves spans a Krylov space of a few dimensions, so a
    cycle that cannot reach its tolerance meets directions that lie in the span of the earlier ones.  The
    solve ends finite, at the accuracy of the arithmetic, and says that it did not converge."""
    need_gpu()
    flush(f"[gpu] exhausted Krylov space {dims}")
    V = int(np.prod(dims))
    x = np.stack(np.unravel_index(np.arange(V), dims), axis=1)
    spin = np.arange(1, 13).reshape(4, 3) + 1j
    wave = [np.exp(2j * math.pi * (x @ (np.array(n) / np.array(dims)))) for n in ((0, 0, 0, 0), (1, 0, 1, 0))]
    b = to_dev((wave[0][:, None, None] + 0.5 * wave[1][:, None, None]) * spin)
    th = torch.zeros((V, 4), dtype=torch.float64, device="cuda")
    with P.Dirac(to_dev(gen.unit_links(dims)), th, dims, 0.11, 1.0, 1.0, 1, (0.0, 0.0, 0.0, 0.0)) as D:
        for method in (P.GCR, P.MIXED_GCR):
            y = torch.zeros_like(b)
            info = D.solve(y, b, method=method, tol=1e-17, restart=24, max_iter=60, raise_on_noconv=False)
            assert torch.isfinite(torch.view_as_real(y)).all() and info.true_rel_res < 1e-13, (method, info.true_rel_res)
