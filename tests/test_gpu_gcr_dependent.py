"""GCR on directions that are nearly dependent but needed.

Free field (unit links, periodic), kappa = 1 / (2 sqrt(10)): on even sites D-hat has the eigenvalues
a - C^2 / a, a = sqrt(10), C the sum of the cosines of the momentum, so the constant wave (C = 4) and the wave
alternating in time (C = 2) are eigenvectors of -6/a and +6/a.  With the weights 1 and 1 + eta of the two, <r, D-hat r>
nearly vanishes: the first step of GCR hardly moves, and the second direction's image lies in the span of the
first up to sin = eta.  That rest is the direction that solves the system in two steps, to about (rounding of the
stored vectors) / eta of the right-hand side.
"""
import math

import numpy as np
import pytest
import torch

import gen
import paper_2502_02490_amd as P
from gpu_util import flush, need_gpu, to_dev

pytestmark = pytest.mark.gpu

DIMS = [(4, 4, 4, 4), (16, 16, 16, 18)]  # chunks of 64 sites over eight wavefronts; one site a thread


def operator(dims):
    V = int(np.prod(dims))
    th = torch.zeros((V, 4), dtype=torch.float64, device="cuda")
    return P.Dirac(to_dev(gen.unit_links(dims)), th, dims, 0.5 / math.sqrt(10.0), 1.0, 1.0, 1, (0.0, 0.0, 0.0, 0.0))


def two_waves(dims, eta):
    x = np.stack(np.unravel_index(np.arange(int(np.prod(dims))), dims), axis=1)
    even = (x.sum(axis=1) % 2 == 0).astype(np.complex128)
    spin = np.arange(1, 13).reshape(4, 3) + 1j
    return ((even * (1.0 + (1.0 + eta) * (-1.0) ** x[:, 0]))[:, None, None] * spin)


# rounding 2^-53 (2^-24, 2^-11, 2^-8) times a few over eta: 1e-8 (3e-3, 5e-2, 5e-2) times a few
CASES = [("f64", 1e-8, 1e-6), ("f32", 2e-5, 5e-2), ("f16", 0.01, 0.3), ("bf16", 0.08, 0.3)]


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("prec,eta,tol", CASES, ids=lambda v: str(v))
def test_nearly_dependent_direction_is_taken(dims, prec, eta, tol):
    need_gpu()
    flush(f"[gpu] nearly dependent direction {dims} {prec}")
    b = to_dev(two_waves(dims, eta))
    kw = dict(method=P.GCR) if prec == "f64" else dict(method=P.MIXED_GCR, inner_prec=prec, inner_tol=0.4 * tol)
    with operator(dims) as D:
        x = torch.zeros_like(b)
        info = D.solve(x, b, tol=tol, restart=8, max_iter=40, raise_on_noconv=False, **kw)
        flush(f"[gpu] single: {info.iters} iterations, {info.restarts} restarts, residual {info.true_rel_res:.2e}")
        assert info.true_rel_res < tol and info.iters <= 4 and info.fell_back == 0
        bs, xs = torch.stack([b, 2.0 * b, -1j * b]), torch.zeros((3,) + b.shape, dtype=b.dtype, device="cuda")
        for inf in P.solve_batched([D], [xs], [bs], 3, tol=tol, restart=8, max_iter=40, **kw)[0]:
            assert inf.true_rel_res < tol and inf.iters <= 4 and inf.fell_back == 0


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
def test_dependent_direction_does_not_stall(dims):
    """Equal weights: <r, D-hat r> = 0 (a breakdown of GCR), and nothing but rounding is left of the second direction.
    It is taken as it is and leads out of the breakdown within the cycle of ten."""
    need_gpu()
    flush(f"[gpu] dependent direction {dims}")
    b = to_dev(two_waves(dims, 0.0))
    with operator(dims) as D:
        x = torch.zeros_like(b)
        info = D.solve(x, b, method=P.GCR, tol=1e-10, restart=10, max_iter=40, raise_on_noconv=False)
        flush(f"[gpu] {info.iters} iterations, {info.restarts} restarts, residual {info.true_rel_res:.2e}")
        assert torch.isfinite(torch.view_as_real(x)).all() and info.true_rel_res < 1e-10


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_unreachable_tolerance_is_reported(prec):
    """A tolerance below the accuracy of FP64: the status says so, whatever the inner precision."""
    need_gpu()
    dims = (4, 4, 4, 4)
    U, th = gen.su3_field(dims, 0.4, 5), gen.u1_field(dims, 0.3, 5)
    b = to_dev(gen.gaussian_spinor(dims, 6))
    kw = dict(method=P.GCR) if prec == "f64" else dict(method=P.MIXED_GCR, inner_prec=prec)
    with P.Dirac(to_dev(U), to_dev(th), dims, 0.12, 1.2, 1.0, -1) as D:
        x = torch.zeros_like(b)
        with pytest.raises(P.DiracError) as err:
            D.solve(x, b, tol=1e-18, restart=24, max_iter=200, **kw)
        assert err.value.status == P._lib.ENOCONV
        info = D.solve(x, b, tol=1e-18, restart=24, max_iter=200, raise_on_noconv=False, **kw)
        assert info.true_rel_res < 1e-13 and info.iters <= 200


@pytest.mark.parametrize("restart,max_iter", [(2, 40), (3, 40), (8, 2)])
def test_correction_at_the_end_of_a_cycle(restart, max_iter):
    """The step that needs its correction is the last or the last but one of a cycle, or the last that max_iter allows."""
    need_gpu()
    dims, eta, tol = DIMS[0], 1e-8, 1e-6
    flush(f"[gpu] correction at the end of a cycle, restart {restart}, max_iter {max_iter}")
    b = to_dev(two_waves(dims, eta))
    with operator(dims) as D:
        x = torch.zeros_like(b)
        info = D.solve(x, b, method=P.GCR, tol=tol, restart=restart, max_iter=max_iter)
        assert info.true_rel_res < tol and info.iters == 2
        xs = torch.zeros((1,) + b.shape, dtype=b.dtype, device="cuda")
        inf = P.solve_batched([D], [xs], [b[None].contiguous()], 1, method=P.GCR, tol=tol, restart=restart, max_iter=max_iter)
        assert inf[0][0].true_rel_res < tol and inf[0][0].iters == 2
