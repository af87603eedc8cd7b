"""The one-workgroup eigensolver on matrices that are not ordinary numbers: a
NaN anywhere is reported, never rotated away, and scales at which the squares of
the entries, but not their cubes, are in range give the scaled result (down to
1e-125: entries below 1e-150 count as zero, which has to be below the rounding).

Against numpy, 1e-14 n of the matrix' norm, as for matrices of ordinary scale."""
import numpy as np
import pytest

from gpu_helpers import to_dev, to_host
from test_gpu_jacobi_small import matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 4, 16, 33, 46, 47, 64, 70])
def test_nan_entries_are_reported(pw, ctx, n):
    """Each pair of the first round (0 and m, k and m - k, n padded to m + 1) and
    some others: no pair's rotation may drop the entry."""
    m = n + n % 2 - 1
    pairs = [(0, m)] + [(k, m - k) for k in range(1, (m + 1) // 2)] + [(0, 1), (0, 0), (n - 1, n - 1)]
    for i, j in [p for p in pairs if max(p) < n][::max(1, len(pairs) // 6)]:
        A = matrix("random", n)
        A[i, j] = A[j, i] = np.nan
        with pytest.raises(pw.PWError) as e:
            ctx.heev(to_dev(np.ascontiguousarray(A.T)))
        assert e.value.status == 7, (i, j)


@pytest.mark.parametrize("scale", [1e-125, 1e-110, 1e110, 1e140])
@pytest.mark.parametrize("n", [2, 3, 24, 45, 46, 47, 64, 70])
def test_scales(pw, ctx, n, scale):
    A = matrix("random", n) * scale
    w, Q = ctx.heev(to_dev(np.ascontiguousarray(A.T)))
    w, Q = to_host(w) / scale, to_host(Q).T
    A = A / scale
    tol = 1e-14 * n * np.linalg.norm(A)
    assert np.abs(w - np.linalg.eigvalsh(A)).max() <= tol
    assert np.linalg.norm(A @ Q - Q * w) <= tol
    assert np.linalg.norm(Q.conj().T @ Q - np.eye(n)) <= 1e-14 * n * np.sqrt(n) + 1e-15
