"""Multigrid passes over node ranges that end around a multiple of a workgroup's
threads: coarse levels of 512, 513, 1024, 1025, 1536 and 1537 nodes on one workgroup.

Bar as in tests/test_gpu_gmg.py: 1e-10 at cg_rtol 1e-13 (FP64), 1e-9 at 1e-12 (FP32 with
refinement)."""
import pytest

from tests.gpu_helpers import compare, run_gpu, run_oracle
from workloads import density_uniform_noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(62, 30), (52, 36), (62, 62), (80, 48), (94, 62), (104, 56)])
@pytest.mark.parametrize("precision,rtol,bar", [(0, 1e-13, 1e-10), (1, 1e-12, 1e-9)])
def test_levels_around_multiples_of_the_threads(gpu, nx, ny, precision, rtol, bar):
    cfg = dict(nx=nx, ny=ny, n_steps=12, n_slices=3, pnorm=8, cg_rtol=rtol, max_iter=20000,
               precision=precision, precond=1)
    rho = density_uniform_noise(nx, ny, nx * ny)
    g = run_gpu(cfg, rho, with_status=True)
    e = compare(g, run_oracle(cfg, rho))
    print(nx, ny, precision, e, g["status"], flush=True)
    assert g["status"]["status"] == 0
    assert max(e.values()) <= bar
