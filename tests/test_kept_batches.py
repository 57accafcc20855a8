"""The device allocations that destroyed batches leave for later ones (CPU): relserve_api.hip linked with a HIP runtime of the test's own
(tests/host/kept_batches.cpp), in which streams run when the test says so, captures refuse what they refuse, and memory is counted."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_11546_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("kept")
    common = ["hipcc", "-O1", "-g", "-std=c++17", "--offload-arch=gfx950", "-fno-gpu-rdc", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = []
    for src in (os.path.join(CSRC, "relserve_api.hip"), os.path.join(ROOT, "tests", "host", "kept_batches.cpp")):
        objs.append(str(tmp / (os.path.basename(src) + ".o")))
        r = subprocess.run([*common, "-x", "hip", "-c", src, "-o", objs[-1]], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
    out = str(tmp / "kept_batches")
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", *objs, "-o", out, "-pthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


@pytest.mark.parametrize("case", ["reuse", "other_stream_behind_default", "default_behind_other_stream", "bounded", "batch_outlives_the_layers",
                                  "destroy_allocates_nothing", "inside_a_capture", "threads"])
def test_kept_allocations(exe, case):
    r = subprocess.run([exe, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout[-500:] + r.stderr[-500:]
