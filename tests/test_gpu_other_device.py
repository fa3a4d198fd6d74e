"""Vectors and gauge fields in the memory of another GPU are copied, not read in place by the kernels."""
import pytest
import torch

import gen
import paper_2502_02490_amd as P
from gpu_util import flush, need_gpu, to_dev

pytestmark = pytest.mark.gpu


def test_memory_of_another_gpu():
    need_gpu()
    if torch.cuda.device_count() < 2:
        pytest.skip("one GPU: no memory of another one")
    dims = (4, 4, 6, 8)
    flush("[gpu] memory of another GPU")
    torch.cuda.set_device(0)
    U, th = to_dev(gen.su3_field(dims, 0.4, 5)), to_dev(gen.u1_field(dims, 0.3, 5))
    net = P.PTC((1, 4, 1))
    net.set_weights([torch.randn(s, dtype=torch.complex64, generator=torch.Generator().manual_seed(k)).numpy()
                     for k, s in enumerate(net.shapes())])
    got = []
    for dev in ("cuda:0", "cuda:1"):
        with P.Dirac(U.to(dev), th.to(dev), dims, 0.12, 1.2, 1.0, -1) as D:
            n = D.native_empty("f32").numel()
            x, g = (torch.randn(n, generator=torch.Generator().manual_seed(k)).to(dev) for k in (7, 8))
            y, gx = torch.zeros_like(x), torch.zeros_like(x)
            torch.cuda.synchronize(dev)
            net.forward(D, y, x)
            net.zero_grad()
            net.backward(D, gx, x, g)
            torch.cuda.synchronize()
            got.append([D.clover().cpu(), y.cpu(), gx.cpu()] + [torch.from_numpy(w) for w in net.get_grad()])
    net.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
