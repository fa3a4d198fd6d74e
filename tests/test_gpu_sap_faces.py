"""Schwarz steps exchange projected faces of the corrections: four blocks along each space direction in turn, so
that the blocks ahead and behind differ, over three cycles (the middle one reads and writes everything)."""
import math

import numpy as np
import pytest
import torch

from gpu_util import Case, flush, need_gpu, rel, to_dev
from oracle import sap as osap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,cstar", [((8, 16, 8, 8), 0), ((8, 8, 16, 8), 0), ((8, 8, 8, 16), 0), ((8, 32, 8, 8), 2)], ids=str)
def test_faces_against_oracle(dims, cstar):
    """3 cycles x 2 colours x 2 steps: 12 FP32 operator applications, whose rounding stays below 1e-5 by far, and
    whose face terms are some tenths of the whole."""
    need_gpu()
    flush(f"[gpu] sap faces {dims} cstar {cstar}")
    c = Case(dims, seed=35, bc_phase=(math.pi, 0.3, 0.0, -0.2), cstar=cstar)
    r = c.spinor(2).astype(np.complex64).astype(np.complex128)
    exp = osap.sap(c.f, r, (4, 4, 4, 4), ncy=3, nmr=2)
    inp = c.D.to_native(to_dev(r.astype(np.complex64)), "f32", "lex")
    out = torch.empty_like(inp)
    c.D.sap(out, inp, ncy=3, nmr=2)
    assert rel(c.D.from_native(out, "f32", "lex").cpu().numpy().astype(np.complex128), exp) < 1e-5
    c.D.close()
