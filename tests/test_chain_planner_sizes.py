"""The chains planned for runs of every size (csrc/chain.cpp, csrc/run.cpp) built
for the host with AddressSanitizer and UndefinedBehaviorSanitizer and executed
symbolically (tests/native/chain_sizes_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_18582_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_chains_of_every_size(tmp_path):
    exe = tmp_path / "chain_sizes_check"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", "chain_sizes_check.cpp")] + \
        [os.path.join(CSRC, f) for f in ("run.cpp", "chain.cpp", "plan.cpp")] + ["-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe), "100"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-3000:])
    assert "failures 0" in r.stdout
    n, past = (int(r.stdout.split(k)[1].split(",")[0]) for k in ("chains ", "with empty steps "))
    assert n > 300 and past > 50
