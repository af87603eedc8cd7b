"""Split targets of the FP64 projector product.  Explicit ones above 2048 act as
2048 (the header's contract), bit for bit, and are not taken for the default;
the default is 512 or 768 for few tiles of short splits and 2048 for 24 tiles, whose
longer splits would leave CUs idle at the end."""
import numpy as np
import pytest

from gpu_helpers import to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


def outputs(pw, ctx, nproj, nb, targets):
    box = (48, 48, 64)
    g, recip, v, oh = problem(box, seed=1)
    rng = np.random.default_rng(2)
    P = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), to_dev(P), rng.uniform(1.0, 2.0, nproj), nb)
    X = to_dev(rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j]))
    H = {}
    for blocks in targets:
        ham.set_tuning({"gemm_blocks": blocks})
        H[blocks] = to_host(ham.apply_h(X))
    return H


def test_explicit_targets_above_the_cap(pw, ctx):
    H = outputs(pw, ctx, 192, 100, (2048, 2049, 4095, 4096, 512))            # 6 tiles
    assert np.array_equal(H[2049], H[2048]) and np.array_equal(H[4095], H[2048])
    assert np.array_equal(H[4096], H[512]) and not np.array_equal(H[512], H[2048])


@pytest.mark.parametrize("nproj,nb,target", [(256, 256, 768), (256, 384, 2048)])   # 16 and 24 tiles
def test_default_of_more_tiles(pw, ctx, nproj, nb, target):
    H = outputs(pw, ctx, nproj, nb, (2048, 4096, 768, 512))
    assert np.array_equal(H[4096], H[target])
    assert not np.array_equal(H[512], H[2048]) and not np.array_equal(H[768], H[2048])
