"""The chain planner (csrc/chain.cpp) built for the host with AddressSanitizer
and UndefinedBehaviorSanitizer (tests/native/chain_check.cpp): every planned
chain, executed symbolically, reads from LDS exactly what its nodes read and
stays inside its arena."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_18582_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_chains_read_what_their_nodes_read(tmp_path):
    exe = tmp_path / "chain_check"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", "chain_check.cpp"), os.path.join(CSRC, "chain.cpp"),
           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe), "150"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-3000:])
    assert "failures 0" in r.stdout
    assert int(r.stdout.split("chains ")[1].split(",")[0]) > 500
