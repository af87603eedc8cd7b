"""bf16 projector products at the edges of their tiles and stages: 1 to 130
projectors (chunks of 32, stages of 64, tiles of 64 and 128), 1 to 65 bands,
plane-wave counts with remainders in either half of a stage and splits that end
on an odd chunk.

Against the oracle on the same rounded input: the projectors (in both products),
their coefficients and the result are rounded to 8 bits, 2^-9 each, in the norm
of a result that the non-local part dominates, so 4 x 2^-9."""
import numpy as np
import pytest

import oracle
from gpu_helpers import frob_err, to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nproj,nb,frac", [(1, 1, 0.05), (31, 2, 0.1), (32, 63, 0.12), (33, 64, 0.14),
                                           (64, 65, 0.16), (65, 5, 0.2), (130, 16, 0.25), (96, 33, 0.22)])
def test_apply(pw, ctx, nproj, nb, frac):
    import torch
    box = (24, 24, 24)
    g, recip, v, oh = problem(box, frac=frac, seed=nproj)
    rng = np.random.default_rng(nproj + 1)
    oh.proj = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
    oh.ekb = 30.0 * rng.uniform(0.5, 1.0, nproj)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), to_dev(oh.proj), oh.ekb, nb, low_prec=True)
    X = rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])
    Xb = pw.to_bf16_pairs(to_dev(X).to(torch.complex64))
    ref = oracle.apply_h(oh, to_host(pw.from_bf16_pairs(Xb)).astype(np.complex128).T).T
    for tuning in ({}, {"nn_tile32": 1}, {"gemm_blocks": 7}):
        ham.set_tuning(tuning)
        out = to_host(pw.from_bf16_pairs(ham.apply_h(Xb, prec="bf16"))).astype(np.complex128)
        assert frob_err(out, ref) < 4 * 2.0 ** -9, tuning
