"""Explicit split targets of the FP64 projector product: above 2048 they act as
2048 (the header's contract), bit for bit, and are not taken for the default."""
import numpy as np
import pytest

from gpu_helpers import to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


def test_explicit_targets_above_the_cap(pw, ctx):
    box, nproj, nb = (48, 48, 64), 192, 100            # 6 tiles: the default aims at 512
    g, recip, v, oh = problem(box, seed=1)
    rng = np.random.default_rng(2)
    P = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), to_dev(P), rng.uniform(1.0, 2.0, nproj), nb)
    X = to_dev(rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j]))
    H = {}
    for blocks in (2048, 2049, 4095, 4096, 512):
        ham.set_tuning({"gemm_blocks": blocks})
        H[blocks] = to_host(ham.apply_h(X))
    assert np.array_equal(H[2049], H[2048]) and np.array_equal(H[4095], H[2048])
    assert np.array_equal(H[4096], H[512]) and not np.array_equal(H[512], H[2048])
