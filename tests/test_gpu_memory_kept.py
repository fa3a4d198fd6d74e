"""Device memory that the library holds beside live contexts, seen from a fresh process: nothing while or after a
program uses one context, at most 1/32 of the device's memory in a program that goes from field to field, and
nothing after release_memory."""
import os
import subprocess
import sys

import pytest

from gpu_util import flush, need_gpu

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import torch
import paper_2502_02490_amd as P

dims = (64, 32, 32, 32)
V = 64 * 32 ** 3
U = torch.eye(3, dtype=torch.complex128, device="cuda").repeat(V, 4, 1, 1)
slack = 256 << 20  # code objects and small buffers; the gauge planes of this lattice take 1,216 MiB
# links and phases of both parities, clover field of both and inverse of one: 96 * 8 + 64, 576 and 576 bytes a site
fields = V // 2 * (2 * (96 * 8 + 64) + 3 * 576)

def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]

def context():
    return P.Dirac(U, None, dims, 0.12, 1.0, 0.0, 1)

start, total = torch.cuda.mem_get_info()
D = context()
print("alive", start - free() - fields, flush=True)
assert start - free() <= fields + slack
D.close()
print("closed", start - free(), flush=True)
assert start - free() <= slack
for _ in range(3):
    context().close()
print("loop", start - free(), flush=True)
assert start - free() <= total // 32 + slack
P.release_memory()
print("released", start - free(), flush=True)
assert start - free() <= slack
"""


def test_memory_beside_live_contexts():
    need_gpu()
    flush("[gpu] memory kept of contexts")
    r = subprocess.run([sys.executable, "-u", "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=90)
    flush(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]


REDUCE = r"""
import torch
import paper_2502_02490_amd as P

dims = (64, 32, 32, 32)
U = torch.eye(3, dtype=torch.complex128, device="cuda").repeat(64 * 32 ** 3, 4, 1, 1)
with P.Dirac(U, None, dims, 0.12, 1.0, 0.0, 1) as D:
    x = D.native_empty("f32")
    x.fill_(0.5)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    d = D.dot(x, x, "f32")
    used = before - torch.cuda.mem_get_info()[0]
    print("work space of the reductions", used, flush=True)
    assert d == 0.25 * 24 * 64 * 32 ** 3
    assert used <= 6 << 20  # two doubles a work-group and the scalars, in allocations of up to 2 MiB
"""


def test_work_space_of_the_reductions():
    need_gpu()
    flush("[gpu] work space of the reductions")
    r = subprocess.run([sys.executable, "-u", "-c", REDUCE], cwd=ROOT, capture_output=True, text=True, timeout=90)
    flush(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
