"""Launch statistics (option kernel_timing) name chains as chains: their launches,
time and work are not in the per-kernel arrays and are in the totals."""
import pytest

import workloads as W
from harness import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", ["resnet20", "mobilenetv2"])
def test_chain_statistics(cfg):
    wl = W.make_workload(cfg, n_inputs=64, n_mutants=20)
    m = run_gpu(wl, kernel_timing=1)[0]
    s = m.stats()
    assert s["chain_launches"] > 0 and s["chain_ms"] > 0 and s["chain_bytes_algorithmic"] > 0
    assert s["gemm_launches"] == sum(s["kernel_launches"]) + s["chain_launches"]
    assert s["gemm_macs_algorithmic"] == sum(s["kernel_macs_algorithmic"]) + s["chain_macs_algorithmic"]
    assert abs(s["ms_gemm"] - sum(s["kernel_ms"]) - s["chain_ms"]) < 1e-3 * s["ms_gemm"]
    layers = run_gpu(wl, kernel_timing=1, fused_paths=0)[0].stats()
    assert layers["chain_launches"] == 0 and layers["chain_ms"] == 0
    # the same work, chains' apart from the layers'
    assert s["gemm_macs_algorithmic"] == layers["gemm_macs_algorithmic"]
    m.set_option("kernel_timing", 0)
    m.run_mutants()
    assert m.stats()["chain_launches"] == 0
