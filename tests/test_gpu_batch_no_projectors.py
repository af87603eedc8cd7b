"""Batches with items that have no projectors (purely local potentials), alone and
beside items that have some: the fused launches against the per-item ones.

Ritz values after three steps agree to 1e-10 of the largest (the same arithmetic
in other orders; FP32 and bf16 filters to 1e-6 and 1e-3, their own rounding)."""
import numpy as np
import pytest

from gpu_helpers import to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-6), ("bf16", 1e-3)])
@pytest.mark.parametrize("nprojs", [(0,), (0, 6, 0), (20, 0)])
def test_items_without_projectors(pw, ctx, nprojs, prec, tol):
    eigs = []
    for mode in ("fused", False):
        hams, xs = [], []
        for i, nproj in enumerate(nprojs):
            box, nb = (24, 25, 24), 12 + i
            g, recip, v, oh = problem(box, seed=i)
            rng = np.random.default_rng(10 + i)
            P = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
            hams.append(pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v),
                                       to_dev(P) if nproj else None,
                                       rng.uniform(0.1, 1.0, nproj) if nproj else None, nb,
                                       low_prec=prec != "fp64"))
            xs.append(to_dev(rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])))
        b = pw.Batch(ctx, hams, xs, degree=4, filter_prec=prec)
        b.chfsi(3, graph=mode)
        eigs.append([to_host(e) for e in b.eig])
        b.close()
    for a, e in zip(*eigs):
        assert np.isfinite(a).all() and np.abs(a - e).max() <= tol * np.abs(e).max()
