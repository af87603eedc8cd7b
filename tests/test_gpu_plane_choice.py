"""The plane kernel that a handle says it runs: every family of boxes and tuning,
among them spheres beyond N/4 and extents that leave no LDS for the two-factor
kernel's exchange buffers, which the general and register kernels then serve."""
import pytest

from gpu_helpers import to_dev
from test_gpu_plane_boxes import problem

pytestmark = pytest.mark.gpu

# box, sphere radius over N, tuning, kernel in FP64 and in FP32
CASES = [
    ((24, 25, 12), 0.25, {}, "k_plane_pq", "k_plane_pq"),
    ((24, 25, 12), 0.30, {}, "k_plane", "k_plane"),           # beyond N/4
    ((48, 48, 12), 0.25, {}, "k_plane_reg", "k_plane_pq"),
    ((48, 48, 12), 0.30, {}, "k_plane_reg", "k_plane_reg"),
    ((48, 48, 12), 0.25, {"reg_plane": 0}, "k_plane_pq", "k_plane_pq"),
    ((36, 36, 12), 0.24, {"plane_variant32": 0}, "k_plane_pq", "k_plane_pq"),
    ((144, 144, 4), 0.24, {}, "k_plane_reg", "k_plane_ls"),
    ((144, 144, 4), 0.24, {"plane_variant32": 0}, "k_plane_reg", "k_plane_pq"),
    ((150, 144, 4), 34.01 / 150, {}, "k_plane", "k_plane_pq"),   # FP64: 160 080 bytes of extent
]


@pytest.mark.parametrize("box,frac,tuning,fp64,fp32", CASES)
def test_plane_kernel(pw, ctx, box, frac, tuning, fp64, fp32):
    g, recip, v, oh = problem(box, frac=frac)
    ham = pw.Hamiltonian(ctx, g, recip, oh.kred, box, to_dev(v), None, None, 2, low_prec=True)
    if tuning:
        ham.set_tuning(tuning)
    assert ham.plane_kernel("fp64") == fp64
    assert ham.plane_kernel("fp32") == ham.plane_kernel("bf16") == fp32
