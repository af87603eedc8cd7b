"""The block eigensolver (n > 64) at the edges of its padding (multiples of 64)
and for the rotation's special cases: zero, diagonal, all diagonal entries
equal, exact multiplets, tiny and large scales.

Against numpy; 1e-14 n of the matrix' norm for eigenvalues, the residual and
orthonormality (each of the about 20 n rotations of a vector rounds to 1e-16,
and the solve stops at off-diagonal entries of 2e-16 n)."""
import numpy as np
import pytest

from gpu_helpers import to_dev, to_host
from test_gpu_jacobi_small import matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["random", "zero", "diagonal", "equal", "multiplets", "tiny", "large"])
@pytest.mark.parametrize("n", [65, 127, 128, 129, 200])
def test_heev_blocks(pw, ctx, n, kind):
    A = matrix(kind, n)
    A = 0.5 * (A + A.conj().T)
    w, Q = ctx.heev(to_dev(np.ascontiguousarray(A.T)))        # column-major
    w, Q = to_host(w), to_host(Q).T
    ref = np.linalg.eigvalsh(A)
    tol = 1e-14 * n * max(np.linalg.norm(A), np.finfo(float).tiny)
    assert np.abs(w - ref).max() <= tol
    assert np.linalg.norm(A @ Q - Q * w) <= tol
    assert np.linalg.norm(Q.conj().T @ Q - np.eye(n)) <= 1e-14 * n * np.sqrt(n) + 1e-15
