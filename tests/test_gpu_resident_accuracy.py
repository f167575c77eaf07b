"""Resident lanes at loose tolerances and near the tightest that FP64 certifies.

Bars: no output further from the oracle than that of the streaming lanes (Jacobi CG,
the general path) at the same cg_rtol; the relative error of Theta, a sum over the
states whose errors can cancel by chance, no larger than that of the states. No step
that starts from an extrapolation is accepted without a round of CG. A tolerance that
the streaming lanes certify is certified."""
import numpy as np
import pytest

from tests.gpu_helpers import rel_max, run_gpu, run_oracle
from workloads import density_branches, density_gaussians, density_uniform_noise

pytestmark = pytest.mark.gpu

STREAM = dict(resident=0)


def _errors(g, o):
    e = {k: rel_max(g[k], o[k]) for k in ("S", "uT", "lam")}
    e["grad"] = float(np.linalg.norm(g["grad"] - o["grad"]) / np.linalg.norm(o["grad"]))
    e["Theta"] = abs(g["Theta"] - o["Theta"]) / o["Theta"]
    return e


@pytest.mark.parametrize("rtol", [1e-3, 1e-5, 1e-7])
@pytest.mark.parametrize("nx,ny,n_slices,n_steps,prop", [(64, 64, 8, 128, 0), (40, 57, 1, 120, 0),
                                                         (48, 48, 6, 96, 1), (64, 48, 6, 96, 2)])
def test_no_less_accurate_than_streaming_lanes(gpu, nx, ny, n_slices, n_steps, prop, rtol):
    cfg = dict(nx=nx, ny=ny, n_steps=n_steps, n_slices=n_slices, propagator=prop, cg_rtol=rtol,
               max_iter=20000)
    rho = density_uniform_noise(nx, ny, nx + ny)
    # a warm cycle of the same design: its fine solves start close to their solutions
    o = run_oracle(cfg, rho)
    guess = None if n_slices == 1 else (o["uT"], o["utheta"], o["lam"])
    o = run_oracle(cfg, rho, guess)
    g = run_gpu(cfg, rho, guess, with_status=True)
    s = run_gpu(dict(cfg, tuning=STREAM), rho, guess, with_status=True)
    eg, es = _errors(g, o), _errors(s, o)
    print(nx, ny, n_slices, prop, rtol, eg, es, g["status"], flush=True)
    assert g["status"]["status"] == s["status"]["status"] == 0
    assert eg.pop("Theta") <= max(es.pop("Theta"), es["S"])
    assert all(eg[k] <= es[k] for k in eg)


@pytest.mark.parametrize("rtol", [1e-2, 1e-4])
def test_extrapolated_starts_take_a_round(gpu, rtol):
    """All but the first three steps of a slice start from an extrapolation."""
    cfg = dict(nx=40, ny=40, n_steps=96, n_slices=4, cg_rtol=rtol, max_iter=20000)
    st = run_gpu(cfg, density_branches(40, 40, 3), with_status=True)["status"]
    print(st, flush=True)
    assert st["status"] == 0
    assert st["cg_iters_fine"] >= st["solves_fine"] - 3 * 4


@pytest.mark.parametrize("nx,n_slices,rho,rtol", [(384, 16, "gauss", 1e-12), (512, 8, "noise", 5e-13)])
def test_certifies_what_streaming_lanes_certify(gpu, nx, n_slices, rho, rtol):
    cfg = dict(nx=nx, ny=nx, n_steps=16 * n_slices, n_slices=n_slices, cg_rtol=rtol,
               max_iter=20000)
    r = density_gaussians(nx, nx, 4) if rho == "gauss" else density_uniform_noise(nx, nx, nx)
    s = run_gpu(dict(cfg, tuning=STREAM), r, with_status=True)["status"]
    g = run_gpu(cfg, r, with_status=True)["status"]
    print(s, g, flush=True)
    assert g["status"] == 0 or s["status"] != 0
