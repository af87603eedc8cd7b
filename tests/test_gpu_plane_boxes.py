"""H*psi (local and kinetic part) in boxes whose N1 and N2 take the two-factor
plane kernels, against the oracle: every factor class of those kernels, odd
and unequal lengths, spheres that reach exactly +-N/4 on both axes, a sphere
that does not fit in N/4 (general kernel), points out of column order, and
enough bands that a workgroup takes several planes.

Tolerances as for the other boxes: 1e-12 in FP64 and 2e-6 in FP32 (the same
sums in another order; FP32 operands and intermediates).
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


def problem(box, frac=0.25, seed=0, shuffle=False):
    """Sphere points inside the ellipsoid with half-axes frac N, a random V."""
    rng = np.random.default_rng(seed)
    r = np.maximum(np.array(box) * frac, 1.0) + 1e-9
    ax = [np.arange(-int(x), int(x) + 1) for x in r]
    g = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    g = g[((g / r) ** 2).sum(1) <= 1.0].astype(np.int32)
    if shuffle:
        g = g[rng.permutation(len(g))]
    recip = 0.3 * np.eye(3)
    v = rng.standard_normal(box[::-1])
    oh = oracle.OracleHam(miller=g, recip=recip, kred=np.array([0.1, -0.2, 0.05]), box=tuple(box),
                          vloc=v, proj=np.zeros((0, len(g)), complex), ekb=np.zeros(0))
    return g, recip, v, oh


# larger factor 8, 10, 12, 16 of N1 and / or N2; odd lengths; N3 outside the register list
BOXES = [(16, 18, 10), (24, 25, 12), (27, 20, 8), (30, 36, 24), (40, 32, 10), (45, 50, 6),
         (48, 64, 6), (54, 60, 5), (72, 80, 4), (81, 90, 4), (100, 96, 4), (108, 100, 3),
         (120, 75, 3), (128, 135, 4), (144, 108, 4), (150, 128, 4), (36, 36, 8), (72, 72, 4),
         (160, 48, 4)]


@pytest.mark.parametrize("box", BOXES, ids=lambda b: "x".join(map(str, b)))
def test_unequal_and_odd_boxes(pw, ctx, box):
    import torch
    g, recip, v, oh = problem(box, seed=sum(box))
    nb = 5
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), None, None, nb, low_prec=True)
    X = np.random.default_rng(1).standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])
    ref = oracle.apply_h(oh, X.T).T
    err = rel_err(to_host(ham.apply_h(to_dev(X))), ref)
    assert err < 1e-12, err
    X32 = to_dev(X).to(torch.complex64)
    ref32 = oracle.apply_h(oh, to_host(X32).astype(np.complex128).T).T
    err = rel_err(to_host(ham.apply_h(X32, prec="fp32")).astype(np.complex128), ref32)
    assert err < 2e-6, err


@pytest.mark.parametrize("box,nb", [((16, 18, 10), 9), ((27, 45, 8), 3), ((36, 36, 12), 40),
                                    ((108, 80, 6), 5), ((72, 72, 4), 7), ((128, 128, 4), 3),
                                    ((75, 120, 4), 2)],
                         ids=lambda b: "x".join(map(str, b)) if isinstance(b, tuple) else str(b))
def test_density_boxes(pw, ctx, box, nb):
    """Density on the same kernels' boxes: more and fewer bands than groups,
    accumulated twice; 1e-12 of the largest value, as for the other boxes."""
    g, recip, v, oh = problem(box, seed=nb)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), None, None, nb)
    X = np.random.default_rng(6).standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])
    w = np.random.default_rng(7).uniform(0.0, 2.0, nb)
    rho = ham.density(to_dev(X), to_dev(w))
    ref = oracle.density(oh, X.T, w)
    assert np.abs(to_host(rho) - ref).max() < 1e-12 * np.abs(ref).max()
    ham.density(to_dev(X[:1]), to_dev(w[:1]), rho=rho, accumulate=True)
    ref = ref + oracle.density(oh, X[:1].T, w[:1])
    assert np.abs(to_host(rho) - ref).max() < 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("frac,shuffle", [(0.4, False), (0.25, True), (0.1, False)])
def test_sphere_forms(pw, ctx, frac, shuffle):
    """A sphere beyond N/4 (general kernel), shuffled points, few columns."""
    box = (30, 24, 20)
    g, recip, v, oh = problem(box, frac=frac, seed=3, shuffle=shuffle)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), None, None, 3)
    X = np.random.default_rng(2).standard_normal((3, len(g), 2)) @ np.array([1.0, 1.0j])
    err = rel_err(to_host(ham.apply_h(to_dev(X))), oracle.apply_h(oh, X.T).T)
    assert err < 1e-12, err


@pytest.mark.parametrize("box,nb", [((32, 30, 27), 150), ((60, 48, 20), 130)])
def test_many_planes_per_workgroup(pw, ctx, box, nb):
    """More (z-plane, band) pairs than resident workgroups: the loop over
    planes and its prefetch; sampled bands against the oracle."""
    g, recip, v, oh = problem(box, seed=4)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), None, None, nb)
    X = np.random.default_rng(5).standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])
    H = to_host(ham.apply_h(to_dev(X)))
    pick = [0, 1, nb // 2, nb - 2, nb - 1]
    err = rel_err(H[pick], oracle.apply_h(oh, X[pick].T).T)
    assert err < 1e-12, err


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_autotune_keeps_the_register_planes(pw, ctx, prec):
    """reg_plane = 0 would select the two-factor planes for H*psi, which the rule
    does by itself, and leave Rayleigh-Ritz above 64 bands the general ones."""
    box, nb = (48, 48, 24), 70
    g, recip, v, oh = problem(box, frac=0.2, seed=3)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), None, None, nb, low_prec=True)
    assert ham.get_tuning()["reg_plane"] == 1
    ham.autotune(prec, nb, reps=1)
    assert ham.get_tuning()["reg_plane"] == 1
