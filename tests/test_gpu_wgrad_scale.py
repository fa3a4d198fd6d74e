"""Weight gradients do not lose accuracy on small gradients: output gradients scaled by 2^-120 (whose lower
mantissa parts lie below the normal BF16 range) give the scaled weight gradients, within the bars
of test_gpu_wgrad.py (its sums and bars are linear in the gradient)."""
import math

import numpy as np
import pytest

import paper_2502_02490_amd as P
from gpu_util import Case, flush, need_gpu
from oracle import ptc as optc
from test_gpu_ptc import to_f32_native
from test_gpu_wgrad import unit_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 4, 6, 8)], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("channels", [(1, 1), (1, 8, 2, 1), (1, 4, 8, 4, 1)], ids=str)
def test_small_output_gradients(dims, channels):
    need_gpu()
    flush(f"[gpu] weight gradients of small gradients {dims} {channels}")
    c = Case(dims, seed=17, bc_phase=(math.pi, 0.3, 0.0, -0.2))
    net = P.PTC(channels)
    try:
        rng = np.random.default_rng(5)
        x = rng.integers(-3, 4, (c.f.V, 4, 3)) + 1j * rng.integers(-3, 4, (c.f.V, 4, 3))
        if len(channels) == 2:  # one layer: the gradient enters in FP32, so any FP32 number is exact
            g = rng.uniform(1, 2, (c.f.V, 4, 3)).astype(np.float32) + 1j * rng.uniform(1, 2, (c.f.V, 4, 3)).astype(np.float32)
        else:
            g = rng.integers(1, 4, (c.f.V, 4, 3)) + 1j * rng.integers(1, 4, (c.f.V, 4, 3))
        ws = unit_weights(channels)
        net.set_weights(ws)
        _, acts = optc.forward(c.f, ws, x)
        _, exact = optc.backward(c.f, ws, acts, g)
        net.zero_grad()
        net.backward(c.D, None, to_f32_native(c.D, x), to_f32_native(c.D, g * 2.0 ** -120))
        got = [w.astype(np.complex128) * 2.0 ** 120 for w in net.get_grad()]
        gl = [g]
        for l in range(len(ws) - 1, -1, -1):
            ng = [np.sqrt((np.abs(v) ** 2).sum(axis=(0, 2))) for v in gl]
            nx = [np.sqrt((np.abs(v) ** 2).sum(axis=(0, 2))) for v in acts[l]]
            bar = 64 * 2.0 ** -24 * np.einsum("cs,dt->cdst", np.array(ng), np.array(nx))
            err = np.abs(got[l] - exact[l]).max(axis=0)
            flush(f"[gpu] layer {l}: {float((err / bar).max()):.3f} of the bar")
            assert (err <= bar).all(), (l, float((err / bar).max()))
            gl = [sum(np.conj(ws[l][0, o, i, 0, 0]) * gl[o] for o in range(len(gl))) for i in range(ws[l].shape[2])]
    finally:
        net.close()
        c.D.close()
