"""The lane trace of resident lanes: times spent waiting on other lanes' flags, and the
window rows per thread and polynomial degree of a lane, by which the tests below know
that each instance of the kernel ran.

Bar: 1e-10 on every output at cg_rtol 1e-13, as in tests/test_gpu_resident.py."""
import numpy as np
import pytest

from tests.gpu_helpers import compare, run_gpu, run_oracle
from workloads import density_uniform_noise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("resident", [-1, 0])
def test_flag_waits_are_told_apart_from_work(gpu, resident):
    """Without a fine lane ahead of it the correction sweep waits for its pass's first
    fine slice from the start: its flag time is about that lane's, and the parts of
    its time add up to its time."""
    cfg = dict(nx=32, ny=32, n_steps=64, n_slices=4, cg_rtol=1e-10, max_iter=20000,
               tuning=dict(phase_timers=1, lead_fine=0, resident=resident))
    tr = run_gpu(cfg, density_uniform_noise(32, 32, 5), with_trace=True)["trace"]
    sweep = next(r for r in tr if r["kind"] == "SWEEP_ADJ")
    first = min(r["step_end_us"][-1] for r in tr if r["kind"] == "F_ADJ")
    total = sweep["step_end_us"][-1] - sweep["start_us"]
    parts = [sweep[k] for k in ("work_us", "barrier_us", "reduce_us", "flag_us")]
    print(first, total, parts, flush=True)
    assert sweep["flag_us"] >= 0.5 * (first - sweep["start_us"])
    assert 0.8 * total <= sum(parts) <= 1.1 * total


# grid, slices, sweep workgroups; window rows per thread of the fine (and batched coarse)
# lanes and of the sweep: tiles cut one way and both, with a ragged last one
ROWS = [(61, 44, 12, 8, 2, 2), (61, 44, 24, 4, 4, 4), (97, 65, 24, 4, 4, 6),
        (61, 130, 12, 8, 4, 4), (90, 74, 24, 4, 6, 6), (127, 96, 24, 8, 6, 6)]


@pytest.mark.parametrize("nx,ny,n_slices,sweep_wgs,fine,sweep", ROWS)
def test_each_number_of_window_rows_runs(gpu, nx, ny, n_slices, sweep_wgs, fine, sweep):
    """Many slices leave a lane few workgroups, and so many window rows per thread."""
    cfg = dict(nx=nx, ny=ny, n_steps=6 * n_slices, n_slices=n_slices, pnorm=8, cg_rtol=1e-13,
               max_iter=20000, tuning=dict(sweep_wgs=sweep_wgs))
    rho = density_uniform_noise(nx, ny, nx + 5 * ny)
    o = run_oracle(cfg, rho)
    guess = (o["uT"], o["utheta"], o["lam"])
    rho = np.clip(rho + 0.02, 0.0, 1.0)
    g = run_gpu(cfg, rho, guess, with_status=True, with_trace=True)
    e = compare(g, run_oracle(cfg, rho, guess))
    shapes = {(r["kind"], r["rows"], r["degree"]) for r in g["trace"]}
    print(nx, ny, n_slices, e, sorted(shapes), g["status"], flush=True)
    rows = {k: {r for q, r, _ in shapes if q == k} for k in ("F_ADJ", "GK_ADJ", "SWEEP_ADJ")}
    assert fine in rows["F_ADJ"] and rows["GK_ADJ"] == {fine} and rows["SWEEP_ADJ"] == {sweep}
    assert g["status"]["status"] == 0
    assert max(e.values()) <= 1e-10


def test_streaming_lanes_have_no_window(gpu):
    cfg = dict(nx=32, ny=32, n_steps=8, n_slices=2, tuning=dict(resident=0))
    tr = run_gpu(cfg, density_uniform_noise(32, 32, 5), with_trace=True)["trace"]
    assert {(r["rows"], r["degree"]) for r in tr} == {(0, 0)}
