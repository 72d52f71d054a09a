"""The shapes of test_turn_tiles_gpu.py still run what they are listed for: tests/host/turn_routes.hip asks the planner.  No GPU."""
import os
import shutil
import subprocess

import pytest

from tests.test_turn_tiles_gpu import SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_shapes_take_the_tiles_they_are_listed_for(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "turn_routes")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-inline-asm", os.path.join(ROOT, "tests", "host", "turn_routes.hip"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, cwd=str(tmp_path))
    assert res.returncode == 0, res.stderr[-4000:]
    calls = [(N, D, V, N - N // 5 if form == "compact" else 0, int(form != "accumulate")) for N, D, V, form, _ in SHAPES]
    out = subprocess.run([exe, *[str(x) for c in calls for x in c]], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr[-2000:]
    for shape, line in zip(SHAPES, out.stdout.strip().split("\n"), strict=True):
        got = dict((k, int(v)) for k, v in (word.split("=") for word in line.split()))
        assert got["turn"] > 0 and all(got[word] for word in shape[4]), (shape, got)
