"""Split-K products A^H B at the edges of their split and reduction rules:
split counts of 1, a few, up to 32 and above (4, 8 and 16 threads to an
element), 64 and 65 columns (threads per element against one ordered sum),
few tiles and many.  Against numpy; 1e-12 of the largest element, as for the
other products (sums of at most 40000 terms in FP64)."""
import numpy as np
import pytest

from gpu_helpers import max_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(8, 16, 31), (8, 16, 40), (1, 1, 300), (8, 16, 1189), (5, 64, 2047),
                                   (5, 65, 2047), (64, 64, 1100), (64, 65, 1100), (70, 3, 40000),
                                   (129, 130, 9000), (400, 500, 700), (20, 200, 16500)])
def test_gemm_cn(pw, ctx, m, n, k):
    rng = np.random.default_rng(m + n + k)
    A = rng.standard_normal((m, k)) + 1j * rng.standard_normal((m, k))   # rows = columns of A
    B = rng.standard_normal((n, k)) + 1j * rng.standard_normal((n, k))
    C = to_host(ctx.gemm_cn(to_dev(A), to_dev(B), alpha=0.5))             # (n, m)
    ref = 0.5 * (B @ A.conj().T)
    assert max_err(C, ref) < 1e-12
    again = to_host(ctx.gemm_cn(to_dev(A), to_dev(B), alpha=0.5))
    assert np.array_equal(C, again)                                        # fixed order of the sums
