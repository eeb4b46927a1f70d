"""What a run launches and where its tensors stand (csrc/run.cpp with
csrc/chain.cpp and csrc/plan.cpp) built for the host with AddressSanitizer and
UndefinedBehaviorSanitizer (tests/native/run_check.cpp): every launch reads
tensors that are computed, stored and not yet overwritten, and chains and the
thin convolution kernel run where they are the faster ones."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_18582_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_runs_read_what_was_computed(tmp_path):
    exe = tmp_path / "run_check"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", "run_check.cpp")] + \
        [os.path.join(CSRC, f) for f in ("run.cpp", "chain.cpp", "plan.cpp")] + ["-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe), "400"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-3000:])
    assert "failures 0" in r.stdout
    assert int(r.stdout.split("chains ")[1].split(",")[0]) > 1000
