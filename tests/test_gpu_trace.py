"""The lane trace of resident lanes: times spent waiting on other lanes' flags."""
import pytest

from tests.gpu_helpers import run_gpu
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
