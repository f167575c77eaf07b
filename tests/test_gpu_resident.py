"""Resident lanes (pt_resident.hip) where their shapes change: one tile and
many, tiles narrower than the halo, ragged last tiles, each number of window
rows per thread, sweep groups of one and of many workgroups, a source that
jumps (the extrapolated starts of the fine steps are then worse than the plain
ones), and solves held to a tolerance near round-off (CG restarts from the true
residual).

Bar: 1e-10 on every output at cg_rtol 1e-13, the bar of the parity tests (the
solves end at a true residual of 1e-13 ||b||, condition numbers stay below 1e3
at these sizes)."""
import numpy as np
import pytest

from tests.gpu_helpers import compare, run_gpu, run_oracle
from workloads import density_uniform_noise

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    c = dict(nx=32, ny=32, n_steps=32, n_slices=4, pnorm=8, cg_rtol=1e-13, max_iter=20000)
    c.update(kw)
    return c


def _check(cfg, rho, bar=1e-10):
    g = run_gpu(cfg, rho, with_status=True)
    e = compare(g, run_oracle(cfg, rho))
    print({k: cfg[k] for k in ("nx", "ny", "n_steps", "n_slices")}, cfg.get("tuning"), e,
          g["status"], flush=True)
    assert g["status"]["status"] == 0
    assert max(e.values()) <= bar


@pytest.mark.parametrize("nx,ny", [(3, 90), (90, 2), (44, 61), (97, 65), (127, 96)])
@pytest.mark.parametrize("rows", [2, 4, 8])
def test_tiles_of_every_row_count(gpu, nx, ny, rows):
    cfg = _cfg(nx=nx, ny=ny, n_steps=24, n_slices=3, tuning=dict(resident_npt_max=rows))
    _check(cfg, density_uniform_noise(nx, ny, nx + 7 * ny))


@pytest.mark.parametrize("wgs", [1, 5, 64])
def test_sweep_groups_of_one_and_of_many_workgroups(gpu, wgs):
    cfg = _cfg(nx=38, ny=29, tuning=dict(sweep_wgs=wgs))
    _check(cfg, density_uniform_noise(38, 29, 3))


def test_source_with_jumps(gpu):
    q = np.where(np.arange(41) % 10 < 5, 1.0, 0.05)
    cfg = _cfg(nx=30, ny=26, n_steps=40, n_slices=2, q=q)
    _check(cfg, density_uniform_noise(30, 26, 4))


def test_restarts_near_round_off(gpu):
    """cg_rtol 2e-16 cannot be certified: every solve restarts from its true
    residual until the cap, reports PT_ENOCONV and keeps a solution that is as
    good as round-off allows."""
    cfg = _cfg(nx=33, ny=30, n_steps=8, n_slices=2, cg_rtol=2e-16, max_iter=300)
    rho = density_uniform_noise(33, 30, 5)
    g = run_gpu(cfg, rho, with_status=True)
    e = compare(g, run_oracle(cfg, rho))
    print(e, g["status"], flush=True)
    assert g["status"]["status"] == -4
    assert max(e.values()) <= 1e-10


@pytest.mark.parametrize("nx,ny,propagator", [(256, 230, 0), (300, 310, 0), (320, 288, 2)])
@pytest.mark.parametrize("warm", [False, True])
def test_grids_that_leave_one_group_beside_the_sweep(gpu, nx, ny, propagator, warm):
    """Grids of which the device holds few groups (two window rows per thread make
    them few already at these sizes): every lane in one queue with the sweeps first and
    last, or one group for all fine and batched coarse lanes. dtau / h^2 <= 610, as above
    condition numbers stay below 1e3."""
    cfg = _cfg(nx=nx, ny=ny, n_steps=12, n_slices=3, t_final=0.018, propagator=propagator,
               tuning=dict(resident_npt_max=2))
    rho = density_uniform_noise(nx, ny, nx)
    ref = run_oracle(cfg, rho)
    guess = None
    if warm:
        guess = (ref["uT"], ref["utheta"], ref["lam"])
        rho = np.clip(rho + 0.02, 0.0, 1.0)
        ref = run_oracle(cfg, rho, guess)
    g = run_gpu(cfg, rho, guess, with_status=True, with_trace=True)
    e = compare(g, ref)
    wgs = {r["kind"]: r["nwg"] for r in g["trace"]}
    print(nx, ny, propagator, warm, e, wgs, g["status"], flush=True)
    assert g["status"]["status"] == 0
    if propagator == 0:
        assert len(set(wgs.values())) == 1
    assert max(e.values()) <= 1e-10


@pytest.mark.parametrize("nx,ny", [(2, 60), (44, 2), (90, 74), (126, 130)])
@pytest.mark.parametrize("tuning", [dict(resident_npt_max=2), dict(resident_npt_max=4),
                                    dict(cm_sweep_wgs=1), dict(resident=0)])
def test_coarse_mesh_lanes(gpu, nx, ny, tuning):
    """Coarse-mesh lanes on every number of window rows, on one workgroup, and in a
    streaming launch; cold and warm (condition numbers as above)."""
    cfg = _cfg(nx=nx, ny=ny, n_steps=16, n_slices=4, propagator=2, cmin=0.5, pc=2.0,
               tuning=tuning)
    rho = density_uniform_noise(nx, ny, nx + 3 * ny)
    _check(cfg, rho)
    o = run_oracle(cfg, rho)
    rho = np.clip(rho + 0.02, 0.0, 1.0)
    g = run_gpu(cfg, rho, (o["uT"], o["utheta"], o["lam"]), with_status=True)
    e = compare(g, run_oracle(cfg, rho, (o["uT"], o["utheta"], o["lam"])))
    print("warm", e, g["status"], flush=True)
    assert g["status"]["status"] == 0
    assert max(e.values()) <= 1e-10


def test_cold_coarse_mesh_sweep_beyond_the_grid_streams(gpu):
    """A cold coarse-mesh sweep that no group of the device holds runs as streaming
    lanes do, with the same bits (two window rows per thread: the device holds
    760 x 760 elements, 770 x 770 no more)."""
    cfg = _cfg(nx=770, ny=770, n_steps=2, n_slices=2, t_final=0.001, cg_rtol=1e-6, propagator=2)
    rho = density_uniform_noise(770, 770, 9)
    a = run_gpu(dict(cfg, tuning=dict(resident_npt_max=2)), rho, with_status=True)
    b = run_gpu(dict(cfg, tuning=dict(resident=0)), rho, with_status=True)
    print(a["status"], b["status"], flush=True)
    assert a["status"]["status"] == b["status"]["status"] == 0
    for k in ("S", "uT", "lam", "grad"):
        assert np.array_equal(a[k], b[k]), k
