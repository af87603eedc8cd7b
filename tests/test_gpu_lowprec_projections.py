"""Projections with FP32 and bf16 operands: however few workgroups a product of few
output tiles is given, its FP32 sums stay as short as the default split makes
them (64 values of the contraction and up) and are added up in FP64.

4095 asks for those splits one by one, 4096 is the default.  The FP32 sums of
both are the same numbers, so only the order of an FP64 sum differs: about
1e-16 before the result is rounded to FP32, which leaves the same FP32 values
but for one in 1e8 (6e-8 each, 3e-10 of the norm of 192 x 192 of them).  Sums
over some times as many values would differ by 5e-8 and more."""
import numpy as np
import pytest

from gpu_helpers import frob_err, to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp32", 1e-9), ("bf16", 1e-6)])
@pytest.mark.parametrize("nproj,nb", [(192, 192), (70, 300), (400, 10)])
def test_few_tiles_keep_the_short_sums(pw, ctx, prec, tol, nproj, nb):
    import torch
    box = (48, 48, 96)
    g, recip, v, oh = problem(box, seed=nproj)
    rng = np.random.default_rng(nb)
    P = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(0.0 * v), to_dev(P),
                         rng.uniform(1e3, 2e3, nproj), nb, low_prec=True)     # kinetic part below 1e-3
    X = to_dev(rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j]))
    X = X.to(torch.complex64) if prec == "fp32" else pw.to_bf16_pairs(X)
    H = {}
    for blocks in (4096, 4095):
        ham.set_tuning({"gemm_blocks": blocks})
        H[blocks] = to_host(ham.apply_h(X, prec=prec).to(torch.complex64 if prec == "fp32" else torch.float32))
    assert np.isfinite(H[4096]).all()
    assert frob_err(H[4096].astype(np.complex128), H[4095].astype(np.complex128)) < tol
