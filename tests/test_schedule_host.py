"""The backward's schedules (csrc/plan.h) under host sanitizers: tests/host/schedule_fuzz.hip walks every
step of the schedule of seeded shapes, and says which orders the shapes of test_schedule_gpu.py take.  No GPU."""
import os
import shutil
import subprocess

import pytest

from tests import schedule_shapes as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def fuzz(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    tmp_path = tmp_path_factory.mktemp("schedule")
    exe = str(tmp_path / "schedule_fuzz")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17",
           "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-sanitize-recover=undefined",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           os.path.join(ROOT, "tests", "host", "schedule_fuzz.hip"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, cwd=str(tmp_path))
    assert res.returncode == 0, res.stderr[-4000:]

    def run(*args):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
        out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, env=env, timeout=300)
        assert out.returncode == 0, (out.stdout + out.stderr)[-4000:]
        return out.stdout
    return run


def orders(fuzz, calls):
    """What each call (N, D, V, compact rows or 0, dW overwritten) runs."""
    lines = fuzz(*[int(x) for c in calls for x in c]).strip().split("\n")
    got = [dict((k, int(v)) for k, v in (word.split("=") for word in line.split())) for line in lines]
    assert len(got) == len(calls)
    for g in got:
        g["varied"] = int(g["least_parts_h"] != g["parts_h"])
    return got


def test_schedules_stay_in_bounds(fuzz):
    assert "iterations ok" in fuzz(600)


@pytest.mark.parametrize("against_forced", [False, True])
def test_gpu_shapes_take_the_orders_they_are_listed_for(fuzz, against_forced):
    calls, wanted = [], []
    for (N, D, V), forms in (S.AGAINST_FORCED if against_forced else S.AGAINST_ORACLE).items():
        for form, want in forms.items():
            calls.append((N, D, V, N - S.n_ignored(N, against_forced) if form == "compact" else 0, form != "accumulate"))
            wanted.append((form, want))
    for call, (form, want), got in zip(calls, wanted, orders(fuzz, calls)):
        short = {k: (got[k], v) for k, v in want.items() if got[k] < v}
        assert not short, (call, form, short, got)


def test_counted_shapes_take_the_routes_they_are_listed_for(fuzz):
    calls, wanted = zip(*[((*shape, 0, form != "accumulate"), (form, want)) for shape, forms in S.COUNTED.items() for form, want in forms.items()])
    for call, (form, want), got in zip(calls, wanted, orders(fuzz, calls)):
        short = {k: (got[k], v) for k, v in want.items() if got[k] < v}
        assert not short, (call, form, short, got)


def test_logit_tiles_are_those_they_are_listed_for(fuzz):
    calls, wanted = zip(*[((N, D, V, N - N // 4 if form == "compact" else 0, 1), (form, want))
                          for (N, D, V), forms in S.LOGIT_TILES.items() for form, want in forms.items()])
    for call, (form, want), got in zip(calls, wanted, orders(fuzz, calls)):
        short = {k: (got[k], v) for k, v in want.items() if got[k] < v}
        assert not short, (call, form, short, got)


def test_drawn_calls_meet_the_orders(fuzz):
    """More than half of the calls of test_random_schedules leave the plan's own tiling, and every kind of order is among them."""
    calls = []
    for case in range(S.N_DRAWN):
        c = S.drawn(case)
        ignored = int(round(c["frac"] * c["N"]))
        bound = c["N"] - ignored + c["slack"]
        calls.append((c["N"], c["D"], c["V"], bound if c["skip"] and bound < c["N"] else 0, not c["accumulate"]))
    got = orders(fuzz, calls)
    assert sum(1 for g in got if g["schedule"] or g["dhidden_blocks"]) * 2 > len(got)
    for what in ("parts_h", "parts_w", "chunks"):
        assert any(g["schedule"] and g[what] > 1 for g in got), what
    assert any(g["schedule"] and c[3] for c, g in zip(calls, got)) and any(g["schedule"] and not c[4] for c, g in zip(calls, got))
