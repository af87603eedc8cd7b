"""The one-workgroup eigensolver at the edges of its two forms (n <= 46 by
position with two copies, above in place): the smallest sizes, odd and even n
around the change, and matrices that test the rotation's special cases: zero,
diagonal, all diagonal entries equal, exact multiplets, tiny and large scales.

Against numpy; 1e-14 n of the matrix' norm for eigenvalues, the residual and
orthonormality (each of the about 7 n rotations of a vector rounds to 1e-16)."""
import numpy as np
import pytest

from gpu_helpers import to_dev, to_host

pytestmark = pytest.mark.gpu


def matrix(kind, n):
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    A = A + A.conj().T
    if kind == "zero":
        return 0.0 * A
    if kind == "diagonal":
        return np.diag(np.diag(A))
    if kind == "equal":
        return A - np.diag(np.diag(A)) + 3.0 * np.eye(n)
    if kind == "multiplets":
        q, _ = np.linalg.qr(A)
        return (q * np.repeat(np.arange(1.0, n + 1), 3)[:n]) @ q.conj().T
    return {"tiny": 1e-30, "large": 1e30}.get(kind, 1.0) * A


@pytest.mark.parametrize("kind", ["random", "zero", "diagonal", "equal", "multiplets", "tiny", "large"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16, 33, 45, 46, 47, 64])
def test_heev(pw, ctx, n, kind):
    A = matrix(kind, n)
    A = 0.5 * (A + A.conj().T)
    w, Q = ctx.heev(to_dev(np.ascontiguousarray(A.T)))        # column-major
    w, Q = to_host(w), to_host(Q).T
    ref = np.linalg.eigvalsh(A)
    tol = 1e-14 * n * max(np.linalg.norm(A), np.finfo(float).tiny)
    assert np.abs(w - ref).max() <= tol
    assert np.linalg.norm(A @ Q - Q * w) <= tol
    assert np.linalg.norm(Q.conj().T @ Q - np.eye(n)) <= 1e-14 * n * np.sqrt(n) + 1e-15
