"""Rayleigh-Ritz in boxes of unequal and unlisted lengths (the two-factor planes up to
96 bands, the general ones above) and on square ones, on both sides of the lines
at 64 and 96 bands.

Against numpy on the oracle's H: 1e-12 of the largest |H| entry's scale for Ritz
values and for H Y, as for H psi; residual norms and orthonormality as closely."""
import numpy as np
import pytest

import oracle
from gpu_helpers import rel_err, to_dev, to_host
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [65, 96, 97, 130])
@pytest.mark.parametrize("box", [(24, 25, 16), (27, 20, 24), (36, 36, 12), (24, 24, 24)],
                         ids=lambda b: "x".join(map(str, b)))
def test_rayleigh_ritz(pw, ctx, box, nb):
    import torch
    g, recip, v, oh = problem(box, seed=nb)
    rng = np.random.default_rng(nb + 1)
    nproj = 20
    oh.proj = rng.standard_normal((nproj, len(g), 2)) @ np.array([1.0, 1.0j]) / len(g) ** 0.5
    oh.ekb = rng.uniform(-1.0, 1.0, nproj)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), to_dev(oh.proj), oh.ekb, nb)
    X = rng.standard_normal((nb, len(g), 2)) @ np.array([1.0, 1.0j])
    Y = to_dev(X)
    HY, eig = torch.empty_like(Y), torch.empty(nb, dtype=torch.float64, device="cuda")
    res = torch.empty_like(eig)
    ham.orthonormalize(Y)
    ham.rayleigh_ritz(Y, HY, eig, res)
    cprj = to_host(ham.cprj(nb))
    Y, HY, eig, res = to_host(Y), to_host(HY), to_host(eig), to_host(res)
    q, _ = np.linalg.qr(X.T)
    hq = oracle.apply_h(oh, q)
    h = q.conj().T @ hq
    scale = np.abs(np.linalg.eigvalsh(h)).max()
    w, z = np.linalg.eigh(0.5 * (h + h.conj().T))
    assert np.abs(eig - w).max() <= 1e-12 * scale
    assert np.linalg.norm(Y.conj() @ Y.T - np.eye(nb)) <= 1e-12 * nb
    assert rel_err(HY, oracle.apply_h(oh, Y.T).T) <= 1e-12
    ref = np.linalg.norm(hq @ z - (q @ z) * w, axis=0)
    assert np.abs(res - ref).max() <= 1e-11 * ref.max()
    assert rel_err(cprj, Y @ oh.proj.conj().T) <= 1e-12
