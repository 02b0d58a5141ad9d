"""What a call leaves behind when it fails, on a pretended device (the library's
host sources compiled with tests/host/call_state.hip in place of the kernels and
of the HIP calls): the counts, the cache and the batch's totals the next call
starts from, what a capturing stream is given, a budget that does not fit, and
work left behind on a stream the caller does not name.  No GPU needed; skipped
when hipcc is absent."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_2009_03254_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("call_state") / "call_state")
    cmd = [HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-ffp-contract=off",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "host", "call_state.hip"),
           *(os.path.join(CSRC, s) for s in ("capi.cpp", "batch_api.cpp", "tables.cpp")), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


@pytest.mark.parametrize("what", ["counts", "cache", "capture", "batch", "budget", "ready"])
def test_after_a_failed_call(exe, what):
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
