"""Weight gradients of the network's matrix-core contraction alone, against the FP64 oracle.

Inputs and output gradients are small integers and the weights are units on the unshifted path, so
every activation and every back-propagated gradient is exact in BF16 and the only rounding left is
that of the transports and of the contraction.  Bar per entry: K u |g_{c,s}| |x_{c',t}| (2-norms over
the lattice, by Cauchy-Schwarz a bound on the sum of the moduli of the terms), u = 2^-24, with K = 64:
13 u from a transport (6 u in an FP32 link with its phase, 7 u in a three-term complex product) times
sqrt(3) for the colour sum, 24 u from a tile's chain of matrix-core sums (six of them at full size,
2 u each for a sum that is not rounded to nearest, doubled for the sum inside an instruction), and at
most 16 u from the additions over tiles.
"""
import math

import numpy as np
import pytest

import paper_2502_02490_amd as P
from gpu_util import Case, flush, need_gpu
from oracle import ptc as optc
from test_gpu_ptc import from_f32_native, to_f32_native

pytestmark = pytest.mark.gpu


def unit_weights(channels):
    """Units (powers of i) on the unshifted path, every input and every output channel connected."""
    ws = []
    for ci, co in zip(channels[:-1], channels[1:]):
        w = np.zeros((9, co, ci, 4, 4), dtype=np.complex128)
        for k in range(max(ci, co)):
            w[0, k % co, k % ci] = 1j ** (k + 1) * np.eye(4)
        ws.append(w)
    return ws


# (4, 8, 8, 16): each XCD's part of a time slice is one block (x1-split tile order); the others take the
# contiguous order, (6, 6, 6, 10) and (2, 2, 2, 2) with a ragged last tile
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 4, 6, 8), (6, 6, 6, 10), (4, 8, 8, 16)], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("channels", [(1, 1), (1, 8, 2, 1), (1, 4, 8, 4, 1), (1, 2, 8, 8, 1)], ids=str)
def test_weight_gradients_exact_activations(dims, channels):
    need_gpu()
    flush(f"[gpu] weight gradients {dims} {channels}")
    c = Case(dims, seed=17, bc_phase=(math.pi, 0.3, 0.0, -0.2))
    net = P.PTC(channels)
    try:
        rng = np.random.default_rng(5)
        x, g = (rng.integers(-3, 4, (c.f.V, 4, 3)) + 1j * rng.integers(-3, 4, (c.f.V, 4, 3)) for _ in range(2))
        ws = unit_weights(channels)
        net.set_weights(ws)
        _, acts = optc.forward(c.f, ws, x)
        _, exact = optc.backward(c.f, ws, acts, g)
        net.zero_grad()
        net.backward(c.D, None, to_f32_native(c.D, x), to_f32_native(c.D, g))
        got = net.get_grad()
        gl = [g]  # gradients at a layer's output, by the unit weights alone
        for l in range(len(ws) - 1, -1, -1):
            ng = [np.sqrt((np.abs(v) ** 2).sum(axis=(0, 2))) for v in gl]
            nx = [np.sqrt((np.abs(v) ** 2).sum(axis=(0, 2))) for v in acts[l]]
            bar = 64 * 2.0 ** -24 * np.einsum("cs,dt->cdst", np.array(ng), np.array(nx))
            err = np.abs(got[l] - exact[l]).max(axis=0)
            assert (err <= bar).all(), (l, float((err / bar).max()))
            gl = [sum(np.conj(ws[l][0, o, i, 0, 0]) * gl[o] for o in range(len(gl))) for i in range(ws[l].shape[2])]
    finally:
        net.close()
        c.D.close()


def test_unaligned_vectors_and_batches():
    """Vectors that are not 16-byte aligned go through copies: the same bits as aligned ones; a minibatch's loss and
    gradient are those of its pairs."""
    import torch

    need_gpu()
    dims, channels = (4, 4, 6, 8), (1, 4, 8, 1)
    flush("[gpu] unaligned network vectors")
    c = Case(dims, seed=18)
    net = P.PTC(channels)
    try:
        net.set_weights(optc.init_weights(channels, seed=2, scale=1.0))
        n = c.D.native_empty("f32").numel()

        def vec(seed, off):
            buf = torch.zeros(n + 4, device="cuda")
            buf[off:off + n] = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")
            return buf[off:off + n]

        got = []
        for off in (0, 1):
            x, g, y, gi = vec(1, off), vec(2, off), vec(3, off), vec(4, off)
            net.forward(c.D, y, x)
            net.zero_grad()
            net.backward(c.D, gi, x, g)
            got.append([y.cpu(), gi.cpu()] + [torch.from_numpy(w) for w in net.get_grad()])
        assert all(torch.equal(a, b) for a, b in zip(*got))
        rs, es = [vec(10 + k, k % 2) for k in range(3)], [vec(20 + k, 0) for k in range(3)]
        losses = [net.loss(c.D, [r], [e]) for r, e in zip(rs, es)]
        ws = net.get_weights()
        loss = net.train_step(c.D, rs, es, 1e-3)
        # the loss of a pair is a sum of FP32 squares accumulated in FP64: the two entry points differ by the FP32
        # rounding of y - e and of its scaled copy, 2^-23 relative each
        assert abs(loss - sum(losses) / 3) <= 2 ** -21 * loss
        grad = net.get_grad()
        net.set_weights(ws)
        with pytest.raises(P.DiracError):  # a zero target: refused, weights unchanged
            net.train_step(c.D, rs, [es[0], torch.zeros_like(es[1]), es[2]], 1e-3)
        assert all(np.array_equal(a, b) for a, b in zip(net.get_weights(), ws))
        net.train_step(c.D, rs, es, 1e-3)
        assert all(np.array_equal(a, b) for a, b in zip(net.get_grad(), grad))
    finally:
        net.close()
        c.D.close()
