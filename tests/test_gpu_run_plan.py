"""Residual networks whose launches the run's plan decides (which convolution
computes its ADD, which nodes share a launch): every order of the nodes gives
the results of the layer-by-layer run (option fused_paths = 0), bit for bit,
and the oracle's."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from harness import LOGIT_TOL, device_inputs, run_gpu

pytestmark = pytest.mark.gpu

ALL_OPS = (W.GF, W.NEB, W.NAI, W.NS, W.WS)


def workload(build, hw, n, n_mutants=24):
    b = W.configs._Builder((hw, hw, 3))
    b.dense(b.gap(build(b, b.conv(0, 16, 3, pad=1))), 10, False)
    w, bb = W.configs._draw_weights(b.nodes, "bf16", 0.05, seed=3)
    model = W.Model("run_plan", "bf16", b.nodes, w, bb)
    muts = W.make_mutants(model, n_mutants, 5, "layer_first", model.weighted_nodes(), ops=ALL_OPS)
    return W.Workload("run_plan", model, W.make_inputs(model, n, "normal"), muts, "")


def check(wl):
    m1, w1, k1, s1 = run_gpu(wl)
    m2, w2, k2, s2 = run_gpu(wl, fused_paths=0)
    assert np.array_equal(w1, w2) and np.array_equal(k1, k2) and s1 == s2
    for mid in [-1] + list(range(wl.mutants.n_mutants)):
        assert np.array_equal(m1.get_logits(mid).cpu().numpy(), m2.get_logits(mid).cpu().numpy()), mid
    ref = O.run_vanilla(O.OracleModel(wl.model), wl.inputs, wl.mutants, keep_logits=[0, 1], mutant_ids=[0, 1])
    scale = np.abs(ref.logits).max()
    for mid, want in ((-1, ref.logits), (0, ref.mutant_logits[0]), (1, ref.mutant_logits[1])):
        assert np.abs(m1.get_logits(mid).cpu().numpy() - want).max() <= LOGIT_TOL["bf16"] * scale, mid
    m1.run_original(device_inputs(wl))
    kb, k3, s3 = m1.run_mutants(noalloc=True)
    assert np.array_equal(kb.cpu().numpy().view(np.uint64), w1) and np.array_equal(k3, k1) and s3 == s1


def projection_block(b, src, c, stride, where):
    """conv, conv, projection, ADD; the projection before, between or after the convolutions."""
    def proj():
        return b.conv(src, c, 1, stride=stride, relu=False)
    p = proj() if where == "before" else None
    x = b.conv(src, c, 3, stride=stride, pad=1)
    p = proj() if where == "between" else p
    x = b.conv(x, c, 3, pad=1, relu=False)
    return b.add(x, proj() if where == "after" else p)


@pytest.mark.parametrize("where", ["before", "between", "after"])
def test_projection_order_layer_by_layer(where):
    # planes of 24 and 12: no chains, convolutions with their ADD and single layers
    wl = workload(lambda b, x: projection_block(b, projection_block(b, x, 32, 2, where), 48, 1, where), 24, 21)
    check(wl)


def wide_sum(b, x):                   # C_in 128: the second convolution runs by itself and computes the sum
    x = b.conv(x, 32, 3, stride=2, pad=1)
    x = b.add(b.conv(b.conv(x, 128, 3, pad=1), 32, 3, pad=1, relu=False), x)
    x = b.dwconv(x, 3, pad=1)
    return b.conv(b.conv(x, 32, 3, pad=1), 32, 3, pad=1)


def unchained_width(b, x):            # 3x3 layers of 24 and 40 channels have no chain of their own
    for c in (24, 40):
        x = b.conv(x, c, 1)
        x = b.add(b.conv(b.conv(x, c, 3, pad=1), c, 3, pad=1, relu=False), x)
        x = b.dwconv(b.conv(x, 2 * c, 1, relu=2), 3, pad=1)
    return x


def mobilenetv2(b, x):                # published widths, expansion 6; fewer repeats and a narrower head
    x = W.configs._inverted_residual(b, x, 1, 16, 1, "")
    for c, n, s in ((24, 2, 1), (32, 3, 2), (64, 2, 2), (96, 2, 1), (160, 2, 2), (320, 1, 1)):
        for k in range(n):
            x = W.configs._inverted_residual(b, x, 6, c, s if k == 0 else 1, "")
    return b.conv(x, 640, 1, relu=2)


@pytest.mark.parametrize("build,hw", [(wide_sum, 16), (wide_sum, 32), (unchained_width, 8), (unchained_width, 16),
                                      (mobilenetv2, 32)])
def test_chains_behind_a_fused_sum(build, hw):
    check(workload(build, hw, 21))
