"""Whole latency-optimal calls (sweep.hip) against the schedule's steps.

CPU: every column program performs the steps' own adds (tests/c/sweep_program.cpp, plan.cpp built
with g++). GPU: the whole call gives the same bits as the same plan run one pass at a time through
trivance_allreduce_emulated_steps_ws, on every launch form that forms.h distinguishes (checked on the
host); other GPU tests compare the whole call and the steps with the oracle."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from gpu_util import forms

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_17254_amd", "csrc")
SIDES = """2 3 4 5 7 8 9 10 16 27 32 64 81 100 128 200 243 256 299 300 729 2x2 3x3 9x9 9x9x9 27x27 3x27
9x27 32x32 16x16 8x8 4x4 8x64 4x8 9x8 5x7 4x4x4 8x8x8 2x3x4 1x9 9x1x8 3x3x3x3""".split()


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_column_programs_perform_the_schedules_adds(tmp_path):
    exe = str(tmp_path / "sweep_program")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    os.path.join(ROOT, "tests", "c", "sweep_program.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe, *SIDES], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert "0 failures" in res.stdout


# (dims, elems, dtype, elements the buffer starts beyond an aligned address, dispatch limit, form and
# launch shape as tests/c/forms.cpp prints them): one, up to four and up to twelve operations a level;
# one, two and four cells to a thread; one tile and several to a workgroup; the widest and narrowest
# tiles, columns that end inside a vector and a segment of less than a tile; one to four dimensions;
# launches split over several dispatches.
CASES = [
    ((2,), 1001, "f32", 0, None, "sweep o1 c2 v1"),
    ((3,), 4099, "f32", 1, None, "steps"),
    ((5,), 3, "f32", 0, None, "sweep o1 c2 v1"),
    ((8,), 70_001, "i32", 3, None, "sweep o4 c2 v64"),
    ((9,), 70_003, "f32", 0, 1024, "sweep o1 c2 v64"),
    ((27,), 33_000, "f32", 0, None, "sweep o1 c2 v32"),
    ((64,), 20_002, "f32", 2, 1024, "sweep o4 c2 v8"),
    ((81,), 40_001, "i32", 0, None, "sweep o1 c4 v16"),
    ((243,), 9001, "f32", 0, None, "sweep o1 c4 v8"),
    ((300,), 5003, "f32", 1, None, "sweep o4 c2 v2"),
    ((729,), 4099, "f32", 0, None, "sweep o1 c4 v4"),
    ((1, 9), 1001, "f32", 0, None, "sweep o1 c2 v1"),
    ((9, 9), 26_215, "i32", 1, None, "sweep o1 c4 v16"),
    ((5, 7), 3001, "f32", 0, None, "sweep o12 c1 v2"),
    ((16, 16), 9001, "f32", 0, 1 << 16, "sweep o12 c1 v1"),
    ((32, 32), 4101, "f32", 3, None, "sweep o4 c1 v1 loop"),
    ((8, 64), 4102, "f32", 0, None, "sweep o12 c1 v1 loop"),
    ((8, 8, 8), 5001, "i32", 0, None, "sweep o12 c1 v1 loop"),
    ((9, 9, 9), 7003, "f32", 1, None, "sweep o1 c4 v4"),
    ((2, 3, 4), 129, "f32", 0, None, "sweep o4 c2 v1"),
    ((3, 3, 3, 3), 2001, "f32", 0, None, "sweep o1 c2 v1"),
    ((32, 32), 500, "f32", 0, None, "sweep o4 c1 v1"),
    ((27, 81), 1030, "i32", 0, None, "sweep o1 c4 v1"),
    ((2000,), 1001, "f32", 0, 1024, "sweep o4 c2 v1"),
    ((2, 2, 2, 2), 1001, "f32", 0, None, "sweep o1 c2 v1"),
    ((4, 7), 20, "f32", 0, None, "sweep o12 c1 v1"),
    # passes above 1 GiB, where the step kernels stream their stores
    ((81,), 1_700_000, "f32", 0, None, "sweep o1 c4 v16"),
    ((64,), 1_100_000, "f32", 0, None, "sweep o4 c2 v8"),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_cases_reach_every_form(tmp_path):
    """The forms that the cases name are the ones that run them, and they meet every compiled kernel
    of sweep.hip."""
    assert forms(tmp_path, [("L", c[0], "natural", f"{c[1]}+{c[3]}") for c in CASES]) == [c[5] for c in CASES]
    seen = {f.rsplit(" v", 1)[0] + (" loop" if "loop" in f else "") for *_, f in CASES}
    assert seen == {"steps", "sweep o1 c2", "sweep o1 c4", "sweep o4 c2", "sweep o4 c1",
                    "sweep o4 c1 loop", "sweep o12 c1", "sweep o12 c1 loop"}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_narrow_tiles_on_aliased_rows_run_step_by_step(tmp_path):
    """2187 ranks leave tiles of 16 bytes, which lose to the steps on rows a multiple of 2 MiB apart:
    only there, on powers of three, and where the steps run on 16-byte vectors."""
    calls = [((27, 81), 1 << 19), ((2187,), 3 << 19), ((9, 9, 9, 3), 1 << 20),  # the steps' side
             ((27, 81), (1 << 19) + 4), ((27, 81), 3 << 18), ((27, 81), f"{1 << 19}+1"),
             ((27, 27), 1 << 19), ((8, 9, 27), 1 << 19)]
    got = forms(tmp_path, [("L", dims, "natural", E) for dims, E in calls])
    assert got[:3] == ["steps"] * 3
    assert [f.split(" ")[0] for f in got[3:]] == ["sweep"] * 5


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'x'.join(map(str, c[0]))}-E{c[1]}-{c[2]}"
                                                      f"-o{c[3]}-l{c[4]}")
def test_whole_call_equals_the_steps(case):
    import torch

    import paper_2602_17254_amd as T

    dims, E, dtype, offset, limit, _ = case
    n = int(np.prod(dims))
    print(f"[sweep] {case}", flush=True)
    plan = T.trivance_plan(dims, "L")
    if limit:
        plan = T.trivance_plan_with_dispatch_limit(plan, limit)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + E)
    if dtype == "f32":
        V = torch.randn(n * E, generator=g, device="cuda")
    else:
        V = torch.randint(-2 ** 31, 2 ** 31 - 1, (n * E,), generator=g, device="cuda",
                          dtype=torch.int32)
    ws = torch.empty(max(16, T.trivance_workspace_bytes(plan, E)), dtype=torch.uint8, device="cuda")
    got = torch.empty(n * E + offset + 64, dtype=V.dtype, device="cuda").fill_(7)
    whole = got[offset:offset + n * E].copy_(V).view(n, E)
    steps = V.view(n, E)
    T.trivance_allreduce_emulated_ws(whole, plan, ws)
    for p in range(plan.num_passes):
        T.trivance_allreduce_emulated_steps_ws(steps, plan, ws, p, p + 1)
    torch.cuda.synchronize()
    assert torch.equal(whole.view(torch.int32), steps.view(torch.int32))
    assert bool((got[:offset] == 7).all()) and bool((got[offset + n * E:] == 7).all())
