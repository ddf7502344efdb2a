"""Whole bandwidth-optimal calls (tile.hip, fold.hip) against the schedule's steps.

CPU: every fold program visits each row once and performs the steps' own adds, and so do the tiles
(tests/c/fold_program.cpp, plan.cpp built with g++). GPU: the whole call gives the same bits as the
same plan run one pass at a time through trivance_allreduce_emulated_steps, on every launch form that
forms.h distinguishes (checked on the host); other GPU tests compare the whole call and the steps with
the oracle."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from gpu_util import forms

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_17254_amd", "csrc")
SIDES = """2 3 4 5 6 7 8 9 10 13 16 25 26 27 28 50 64 81 100 128 200 243 256 299 300 729 2x2 3x3 3x27
9x27 27x27 5x7 4x8 9x8 8x64 32x32 16x16 4x4x4 9x9x9 9x9x3 8x8x8 2x2x2 16x16x16 2x3x4 3x5x7x4 1x9
9x1x8 10x11x12 16x18x20 5x6x7x8 6561""".split()


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_fold_programs_perform_the_schedules_adds(tmp_path):
    exe = str(tmp_path / "fold_program")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    os.path.join(ROOT, "tests", "c", "fold_program.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe, *SIDES], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    assert "0 failures" in res.stdout


def test_plans_do_not_write_every_cut():
    """The fold programs are written once per plan, for the cut chosen by counting. Best of 20 plans
    (on a machine where these take 20 to 90 us; with a program written for every cut they took 750
    to 1100 us): the bound lies a factor of three or more from both."""
    import time

    import paper_2602_17254_amd as T

    for dims in ((6561,), (16, 18, 20), (10, 11, 12), (5, 6, 7, 8)):
        best = 1.0
        for _ in range(20):
            t0 = time.perf_counter()
            T.trivance_plan(dims, "B")
            best = min(best, time.perf_counter() - t0)
        assert best < 300e-6, f"{dims}: {best * 1e6:.0f} us"


# (dims, elems, dtype, placement, elements the buffer starts beyond an aligned address, dispatch
# limit, form and launch shape as tests/c/forms.cpp prints them). Small calls in local memory (one, two,
# four and eight cells to a thread); tiles of four and of sixteen waves, narrow and wide, and a wave per
# tile, each in one launch and in two (192 MiB and more) and with the programs of all collectives in one
# launch and in a launch each; a tail of 1 to 3 columns, segments of less than a tile, rows that start
# inside a cache line, and launches split over several dispatches.
CASES = [
    ((2,), 257, "f32", "natural", 0, None, "tile c1 v1"),
    ((8,), 1, "f32", "natural", 0, None, "tile c1 v1"),
    ((7,), 524_291, "i32", "natural", 1, None, "tile c1 v64"),
    ((5, 7), 255, "f32", "natural", 3, None, "tile c1 v1"),
    ((1, 9), 3001, "f32", "natural", 0, None, "tile c1 v1"),
    ((27, 27), 4098, "f32", "natural", 0, 1024, "tile c2 v2"),
    ((243,), 16_389, "f32", "natural", 2, None, "tile c2 v8"),
    ((32, 32), 16_386, "i32", "natural", 0, None, "fold w16 v16 one"),
    ((16, 16, 16), 259, "f32", "natural", 0, None, "tile c4 v1"),
    ((16, 16, 16), 4096, "i32", "natural", 0, None, "tile c8 v2"),
    ((16, 16, 16), 4099, "f32", "natural", 2, None, "fold w16 v4 one"),
    ((9, 9, 9), 10_001, "f32", "schedule", 0, None, "fold w16 v8 one"),
    ((27,), 100_003, "i32", "natural", 1, None, "tile c1 v32"),
    ((20, 20, 20), 70, "f32", "natural", 0, None, "tile c8 v1"),
    ((300,), 20_481, "f32", "natural", 0, 1024, "tile c2 v4"),
    ((243,), 40_005, "f32", "natural", 0, 1 << 16, "fold w16 v32 one"),
    ((9, 9, 9), 4100, "f32", "schedule", 0, 1024, "tile c2 v2"),
    ((8, 64), 5001, "f32", "natural", 0, None, "tile c1 v2"),
    ((3, 5, 7, 4), 6001, "f32", "natural", 0, None, "tile c1 v2"),
    ((3,), 17_000_001, "f32", "natural", 0, None, "fold w1 v64 spread"),
    ((4, 4, 4), 786_436, "i32", "natural", 0, 1 << 20, "fold w1 v64 spread"),
    ((3, 27), 640_007, "f32", "schedule", 1, None, "fold w1 v64 spread"),
    ((243,), 262_145, "f32", "natural", 0, None, "fold w16 v64 spread"),
    ((32, 32), 65_537, "f32", "natural", 3, None, "fold w16 v64 spread"),
    ((50,), 130_001, "i32", "natural", 0, 1 << 16, "fold w4 v64 one"),
    ((27,), 400_003, "f32", "natural", 1, None, "fold w4 v64 one"),
    ((134,), 50_001, "f32", "natural", 0, None, "fold w4 v32 one"),
    ((134,), 400_001, "i32", "natural", 2, None, "fold w4 v64 spread"),
    ((2, 2, 2, 2), 400_002, "f32", "natural", 0, None, "fold w4 v64 one"),
    ((20,), 540_003, "i32", "natural", 3, None, "fold w1 v64 one"),
    ((27,), 540_004, "f32", "natural", 0, 1 << 16, "fold w1 v64 one"),
    ((3, 3, 2, 2), 540_001, "f32", "natural", 0, None, "fold w1 v64 one"),
    ((10, 11, 12), 20_001, "f32", "natural", 0, 1024, "fold w16 v16 one per-collective"),
    ((10, 11, 12), 50_003, "i32", "natural", 1, None, "fold w16 v32 spread per-collective"),
    ((10, 11, 12), 540_002, "f32", "natural", 0, None, "fold w1 v64 spread per-collective"),
    ((5, 6, 7, 8), 4500, "f32", "natural", 0, None, "fold w16 v4 one per-collective"),
    ((2,), 26_000_002, "f32", "natural", 1, None, "fold w1 v64 one"),
    # passes above 1 GiB, where the step kernels stream their stores
    ((243,), 1_400_000, "f32", "natural", 0, None, "fold w1 v64 spread"),
    ((64,), 4_200_000, "f32", "natural", 0, None, "fold w1 v64 spread"),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_cases_reach_every_form(tmp_path):
    """The forms that the cases name are the ones that run them, so that a limit that moves later
    takes no case along unseen; and the cases meet every compiled kernel of tile.hip and fold.hip."""
    assert forms(tmp_path, [("B", c[0], c[3], f"{c[1]}+{c[4]}") for c in CASES]) == [c[6] for c in CASES]
    seen = {c[6] for c in CASES}
    assert {f.split(" v")[0] for f in seen if f.startswith("tile")} == {f"tile c{c}" for c in (1, 2, 4, 8)}
    for waves in (1, 4, 16):
        for launches in ("one", "spread"):
            assert any(f.startswith(f"fold w{waves} ") and launches in f for f in seen)
    for waves in (1, 16):
        assert any(f.startswith(f"fold w{waves} ") and "per-collective" in f for f in seen)
    # more columns than the block index counts (880 GB)
    assert forms(tmp_path, [("B", (6561,), "natural", 1 << 25)]) == ["steps"]
    # tiles at their narrowest and widest
    assert {"fold w4 v32 one", "fold w4 v64 one", "fold w16 v4 one", "fold w16 v64 spread"} <= seen


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_two_and_three_ranks_spread_only_from_cached_rows(tmp_path):
    """On two ranks, and on three whose rows exceed the last-level cache, fold and spread lose to
    the steps; one launch does not."""
    row = 1 << 26  # elements that fill the 256 MiB cache
    calls = [((2,), row // 2), ((2,), 3 * row), ((2, 1), row), ((3,), row + 1), ((1, 3), 2 * row),
             ((3,), row), ((3,), 17_000_000), ((4,), 2 * row), ((2, 2), row)]
    got = forms(tmp_path, [("B", dims, "natural", E) for dims, E in calls])
    assert got == ["fold w1 v64 one"] * 5 + ["fold w1 v64 spread"] * 4


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'x'.join(map(str, c[0]))}-E{c[1]}-{c[2]}"
                                                      f"-{c[3]}-o{c[4]}-l{c[5]}")
def test_whole_call_equals_the_steps(case):
    import torch

    import paper_2602_17254_amd as T

    dims, E, dtype, placement, offset, limit, _ = case
    n = int(np.prod(dims))
    print(f"[fold] {case}", flush=True)
    plan = T.trivance_plan(dims, "B", placement)
    if limit:
        plan = T.trivance_plan_with_dispatch_limit(plan, limit)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + E)
    if dtype == "f32":
        V = torch.randn(n * E, generator=g, device="cuda")
    else:
        V = torch.randint(-2 ** 31, 2 ** 31 - 1, (n * E,), generator=g, device="cuda",
                          dtype=torch.int32)
    got = torch.empty(n * E + offset + 64, dtype=V.dtype, device="cuda").fill_(7)
    whole = got[offset:offset + n * E].copy_(V).view(n, E)
    steps = V.view(n, E)
    T.trivance_allreduce_emulated(whole, plan)
    for p in range(plan.num_passes):
        T.trivance_allreduce_emulated_steps(steps, plan, p, p + 1)
    torch.cuda.synchronize()
    assert torch.equal(whole.view(torch.int32), steps.view(torch.int32))
    assert bool((got[:offset] == 7).all()) and bool((got[offset + n * E:] == 7).all())
