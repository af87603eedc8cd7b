"""H*psi with few projectors (projections without partials, P C added by the
column kernel) at the edges of its rule: 1, 3, 4, 5, 16 projectors against 17
(general products), 64 bands against 65, npw not a multiple of a workgroup,
points out of column order, the overlap option, and the filter's recurrence.
Against the oracle, 1e-12 as for every FP64 H*psi."""
import numpy as np
import pytest

import oracle
from gpu_helpers import rel_err, to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


def handle(pw, ctx, box, nproj, nb, shuffle=False):
    g, recip, v, oh = problem(box, frac=0.2, seed=nproj, shuffle=shuffle)
    rng = np.random.default_rng(nproj + 1)
    oh.proj = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
    oh.ekb = rng.uniform(-1.0, 1.0, nproj)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), to_dev(oh.proj), oh.ekb, nb)
    X = rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])
    return ham, oh, X


@pytest.mark.parametrize("nproj,nb", [(1, 1), (3, 2), (4, 7), (5, 3), (8, 64), (8, 65), (16, 5), (17, 5)])
def test_apply(pw, ctx, nproj, nb):
    ham, oh, X = handle(pw, ctx, (24, 25, 30), nproj, nb)
    ref = oracle.apply_h(oh, X.T).T
    assert rel_err(to_host(ham.apply_h(to_dev(X))), ref) < 1e-12


def test_shuffled_overlap_and_filter(pw, ctx):
    ham, oh, X = handle(pw, ctx, (20, 24, 32), 6, 9, shuffle=True)
    ref = oracle.apply_h(oh, X.T).T
    H = to_host(ham.apply_h(to_dev(X)))
    assert rel_err(H, ref) < 1e-12
    ctx.set_overlap(True)
    try:
        assert np.array_equal(to_host(ham.apply_h(to_dev(X))), H)
    finally:
        ctx.set_overlap(False)
    Y = to_dev(X).clone()
    ham.cheb_filter(Y, 5, 1.0, 80.0, -3.0)
    assert rel_err(to_host(Y), oracle.cheb_filter(oh, X.T, 5, 1.0, 80.0, -3.0).T) < 1e-10
