"""The one-workgroup eigensolver on matrices that are not ordinary numbers: a
NaN anywhere is reported, never rotated away."""
import numpy as np
import pytest

from gpu_helpers import to_dev
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
