"""tests/host/fused_cuts.hip under host sanitizers: parts, items and planes of the backwards at D = 64 and 128.  No GPU."""
import os
import shutil
import subprocess

import pytest

from tests.test_fused_backward_gpu import FORMS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cuts(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    tmp_path = tmp_path_factory.mktemp("fused")
    exe = str(tmp_path / "fused_cuts")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-unused-command-line-argument", os.path.join(ROOT, "tests", "host", "fused_cuts.hip"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, cwd=str(tmp_path))
    assert res.returncode == 0, res.stderr[-4000:]

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=300, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
        assert out.returncode == 0, (out.stdout + out.stderr)[-3000:]
        return out.stdout
    return run


def test_parts_cover_and_planes_fit(cuts):
    assert " 0 failures" in cuts()


def test_gpu_shapes_take_the_cuts_they_are_listed_for(cuts):
    got = [tuple(int(x) for x in line.split()) for line in cuts(*[x for f in FORMS for x in f[:3]]).strip().split("\n")]
    for shape, words in zip(FORMS, got, strict=True):
        assert words == (1, *shape[4]), (shape, words)
    # both kernels of either hidden size with every form of a call, and every cut
    for D in (64, 128):
        for shared in (0, 1):
            assert {f[3] for f in FORMS if f[1] == D and f[4][0] == shared} >= ({"accumulate", "variants", "mean", "shard"} if shared == 0 else {"variants", "shard"})
            assert {f[4][1:] for f in FORMS if f[1] == D and f[4][0] == shared} >= {(0, 1), (1, 0), (1, 1)}
