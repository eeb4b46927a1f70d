"""Chains whose convolutions' reductions fill an instance's k steps, or leave
some of them empty (conv16 in k_chain.hip): every number of steps of 1 x 1
filters, full and with a remainder, and every width of 3 x 3 filters, give the
layer-by-layer run's results bit for bit (option fused_paths = 0)."""
import numpy as np
import pytest

import workloads as W
from harness import run_gpu

pytestmark = pytest.mark.gpu


def check(build, hw, n):
    b = W.configs._Builder((hw, hw, 3))
    b.dense(b.gap(build(b)), 10, False)
    w, bb = W.configs._draw_weights(b.nodes, "bf16", 0.05, seed=3)
    model = W.Model("chain_steps", "bf16", b.nodes, w, bb)
    muts = W.make_mutants(model, 6, 4, "layer_first", model.weighted_nodes(), ops=(W.GF, W.NEB, W.NAI, W.NS, W.WS))
    wl = W.Workload("chain_steps", model, W.make_inputs(model, n, "normal"), muts, "")
    m1, w1, k1, s1 = run_gpu(wl)
    m2, w2, k2, s2 = run_gpu(wl, fused_paths=0)
    assert m1.stats()["launches"] < m2.stats()["launches"]          # no ADD: chains ran
    assert np.array_equal(w1, w2) and np.array_equal(k1, k2) and s1 == s2
    for mid in range(-1, 6):
        assert np.array_equal(m1.get_logits(mid).cpu().numpy(), m2.get_logits(mid).cpu().numpy()), mid


@pytest.mark.parametrize("c", [32 * s - r for s in range(1, 13) for r in (0, 24)])
def test_1x1(c):
    # tiles of 16 output channels: whole, and a half one
    check(lambda b: b.conv(b.conv(b.conv(0, c, 3, pad=1), 64, 1, relu=2), 24, 1), 4, 19)


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("c", [8, 16, 24, 32])
def test_3x3(c, stride):
    check(lambda b: b.conv(b.conv(b.conv(0, c, 3, pad=1), 48, 3, pad=1, stride=stride), 16, 1), 8, 19)
