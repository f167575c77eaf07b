"""The planner of resident lanes (csrc/pt_plan.h) on the host: a launch that it
accepts has to fit the device."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GRID = 256   # workgroups of the device
F_PRI, GK_PRI, SWEEP_PRI, COLD_PRI = 0, 1, 2, 3
CM_GK_PRI, CM_SWEEP_PRI = 8, 9


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(lines) -> the planner's answers, a list of numbers per line."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_probe")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", f"{rocm}/include",
                    os.path.join(ROOT, "tests", "plan_probe.cpp"), "-o", exe], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", text=True, check=True,
                             capture_output=True).stdout
        return [[int(x) for x in l.split()] for l in out.splitlines()]
    return run


def lane(kind, count, latency=0, fixed=0, lead=-1, weight=1.0):
    return f"{kind} {count} 0 1 {weight} {latency} 0 {fixed} {lead}"


def plan(nx, ny, Ntau, lanes, M=16, rows=8, sweep_wgs=64, share=1, cm=0):
    return " ".join([f"plan {nx} {ny} {Ntau} {M} {GRID} {rows} {sweep_wgs} {share} {cm}", *lanes])


def plan_workgroups(answer):
    return sum(answer[3 + 6 * k] * answer[4 + 6 * k] for k in range((len(answer) - 3) // 6))


def test_a_sweep_alone_beyond_the_grid_is_not_resident(ask):
    """The cold coarse-mesh sweep is the only lane of its launch: on grids that
    need more workgroups than the device holds it has to stream."""
    sizes = [256, 768, 1024, 1400, 1500, 1600, 2000, 4000]
    got = ask([plan(n, n, 8, [lane(CM_SWEEP_PRI, 1, latency=1, fixed=24)], cm=1) for n in sizes])
    for n, a in zip(sizes, got):
        assert a[0] == (n <= 1400), (n, a)
        assert not a[0] or plan_workgroups(a) <= GRID, (n, a)


def test_accepted_plans_fit_the_device(ask):
    rng = random.Random(5)
    lines = []
    for _ in range(1500):
        nx, ny = (int(2 ** rng.uniform(0, 11)) for _ in range(2))
        Ntau, M = rng.choice([1, 2, 3, 8, 32, 400]), rng.choice([1, 4, 16])
        prop, warm = rng.randrange(3), rng.randrange(2)
        lead = rng.randrange(2) and Ntau > 1 and prop != 1
        kw = dict(rows=rng.choice([1, 2, 4, 8]), sweep_wgs=rng.choice([1, 40, 64, 300]),
                  share=rng.randrange(2), cm=int(prop == 2 and Ntau > 1))
        if prop == 2:
            nx, ny = 2 * nx, 2 * ny
        lanes = [lane(F_PRI, Ntau - 1 if lead else Ntau, weight=M)]
        if prop != 1 and Ntau > 1:
            if warm:
                lanes.append(lane(CM_GK_PRI if prop == 2 else GK_PRI, Ntau - 1, weight=4.0))
            elif prop == 0:
                lanes.append(lane(COLD_PRI, 1, latency=1))
            sweep = CM_SWEEP_PRI if prop == 2 else SWEEP_PRI
            lanes.append(lane(sweep, 1, latency=1, fixed=24 if prop == 2 else 0,
                              lead=F_PRI if lead else -1))
        lines.append(plan(nx, ny, Ntau, lanes, M=M, **kw))
    got = ask(lines)
    assert sum(a[0] for a in got) > 500
    for l, a in zip(lines, got):
        assert not a[0] or 0 < plan_workgroups(a) <= GRID, (l, a)


def test_coarse_mesh_degree_does_not_depend_on_the_size(ask):
    sizes = [4, 16, 32, 48, 64, 94, 96, 98, 100, 128, 160, 200, 256, 400]
    got = ask([plan(n, n, 8, [lane(CM_SWEEP_PRI, 1, latency=1, fixed=24)], cm=1) for n in sizes])
    assert {n: a[7] for n, a in zip(sizes, got)} == {n: 4 for n in sizes}
