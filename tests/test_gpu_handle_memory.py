"""Device memory of a low-precision handle: of the projectors it keeps their two
three-term copies (12 bytes an entry each) and no other form."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


def test_projector_copies(pw, ctx):
    import torch
    box, nproj = (48, 48, 64), 2000
    g, recip, v, oh = problem(box, seed=1)
    P = torch.zeros((nproj, len(g)), dtype=torch.complex128, device="cuda")
    V, held = to_dev(v), []
    for low in (False, True):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, V, P, np.ones(nproj), 1, low_prec=low)
        held.append(before - torch.cuda.mem_get_info()[0])
        del ham
    per = (held[1] - held[0]) / P.numel()     # 8 more with a complex64 copy; the rest is a few MB
    assert 24.0 <= per <= 28.0, per
