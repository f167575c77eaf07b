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
        assert a[0] or not a[1], (l, a)   # what is refused asks for no shared queue


def test_coarse_mesh_degree_does_not_depend_on_the_size(ask):
    sizes = [4, 16, 32, 48, 64, 94, 96, 98, 100, 128, 160, 200, 256, 400]
    got = ask([plan(n, n, 8, [lane(CM_SWEEP_PRI, 1, latency=1, fixed=24)], cm=1) for n in sizes])
    assert {n: a[7] for n, a in zip(sizes, got)} == {n: 4 for n in sizes}


THREADS, RIM = 512, 2


def rim_cells_lost(W, HN, tw, th, deg, nr):
    """Cells around the windows of a shape's tiles that lie in the grid and have an
    index beyond what the threads hold: the rows above and below first, then the two
    columns beside the rows, in turn (the kernel's order)."""
    TX, TY = -(-W // tw), -(-HN // th)
    hx, hy = (deg + 1 if TX > 1 else 0), (deg + 1 if TY > 1 else 0)
    wc, wr = tw + 2 * hx, th + 2 * hy
    rows = min(THREADS // wc, -(-wr // nr)) * nr
    sz = wc + 2
    lost = 0
    for ty in {0, TY // 2, TY - 1}:
        for tx in {0, TX // 2, TX - 1}:
            for e in range(RIM * THREADS, 2 * sz + 2 * rows):
                if e < 2 * sz:
                    cx, cy = e % sz, 0 if e < sz else rows + 1
                else:
                    cx, cy = (sz - 1 if e & 1 else 0), 1 + ((e - 2 * sz) >> 1)
                gx, gy = tx * tw - hx - 1 + cx, ty * th - hy - 1 + cy
                lost += 0 <= gx < W and 0 <= gy < HN and cy <= wr + 1
    return lost


def test_windows_that_fit_lose_no_cell_of_their_rim(ask):
    rng = random.Random(11)
    cases = [(4, 1300, 1, 600, 1, 6), (2, 1300, 1, 1000, 0, 6), (9, 1300, 3, 600, 0, 6),
             (4, 1300, 4, 600, 1, 6), (300, 2, 300, 2, 3, 2), (900, 3, 450, 3, 3, 6)]
    for _ in range(3000):
        W, HN = (int(2 ** rng.uniform(1, 11)) for _ in range(2))
        tw = max(1, int(W / 2 ** rng.uniform(0, 8)))
        th = max(1, int(HN / 2 ** rng.uniform(0, 8)))
        cases.append((W, HN, tw, th, rng.randrange(9), rng.choice([2, 4, 6])))
    got = ask(["window " + " ".join(map(str, c)) for c in cases])
    assert [g[0] for g in got[:6]] == [0, 0, 0, 1, 1, 1]
    assert sum(g[0] for g in got) > 500
    for c, g in zip(cases, got):
        if g[0]:
            assert rim_cells_lost(*c) == 0, c
            assert g[1] <= 160 * 1024 - 1024, c
    assert rim_cells_lost(*cases[0]) > 0 and rim_cells_lost(*cases[2]) > 0
