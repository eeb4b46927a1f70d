"""Chains of small bf16 layers in one launch (k_chain.hip) give exactly the
layer-by-layer kernels' results (option fused_paths = 0), bit for bit."""
import numpy as np
import pytest

import workloads as W
from harness import run_gpu
from paper_2607_18582_amd import Mure

pytestmark = pytest.mark.gpu

ALL_OPS = (W.GF, W.NEB, W.NAI, W.NS, W.WS)


def same(wl, **opt):
    m1, w1, k1, s1 = run_gpu(wl, **opt)
    m2, w2, k2, s2 = run_gpu(wl, fused_paths=0, **opt)
    assert m1.stats()["launches"] < m2.stats()["launches"]          # chains did run
    assert np.array_equal(w1, w2) and np.array_equal(k1, k2) and s1 == s2
    for mid in [-1] + list(range(wl.mutants.n_mutants)):
        assert np.array_equal(m1.get_logits(mid).cpu().numpy(), m2.get_logits(mid).cpu().numpy()), mid


@pytest.mark.parametrize("vanilla", [0, 1])
@pytest.mark.parametrize("n", [1, 7, 131])                          # fewer images than a block takes; remainders
@pytest.mark.parametrize("cfg", ["resnet20", "mobilenetv2"])
def test_chains_equal_layers(cfg, n, vanilla):
    same(W.make_workload(cfg, n_inputs=n, n_mutants=40, ops=ALL_OPS), vanilla=vanilla)


def graph(name):
    b = W.configs._Builder((16, 16, 3))
    x = b.conv(0, 16, 3, pad=1)
    if name == "odd":                 # an activated conv before its ADD, dw without one, 48 and 24 channels
        a = b.conv(x, 16, 3, pad=1)
        x = b.add(b.conv(a, 16, 3, pad=1, relu=True), x, relu=False)
        x = b.conv(x, 48, 1, relu=False)
        x = b.dwconv(x, 3, pad=1, relu=0)
        x = b.conv(x, 32, 3, pad=1)                                  # halo order, C_in 48
        x = b.conv(x, 24, 1, relu=2)
        x = b.dwconv(x, 3, stride=2, pad=1, relu=1)
        x = b.conv(x, 64, 1)
    else:                             # 64 channels at 8 x 8 and below, more than 64 of them changed at once
        x = b.conv(x, 32, 3, stride=2, pad=1)
        x = b.conv(x, 64, 3, pad=1)
        y = b.conv(x, 64, 3, pad=1)
        x = b.add(b.conv(y, 64, 3, pad=1, relu=False), x)
        x = b.conv(x, 128, 1, relu=2)
        x = b.dwconv(x, 3, stride=2, pad=1)
        x = b.conv(x, 40, 1, relu=False)
    b.dense(b.gap(x), 10, False)
    w, bb = W.configs._draw_weights(b.nodes, "bf16", 0.05, seed=3)
    return W.Model(name, "bf16", b.nodes, w, bb)


@pytest.mark.parametrize("name,k", [("odd", 5), ("wide", 5), ("wide", 90)])
def test_chains_of_other_shapes_equal_layers(name, k):
    model = graph(name)
    layers = model.weighted_nodes()
    if k > 64:                        # every mutant changes most of the 128-channel expansion
        layers = [i for i in layers if model.nodes[i].c_out == 128 and model.nodes[i].kind == W.CONV2D]
    muts = W.make_mutants(model, 24, k, "layer_first", layers, ops=ALL_OPS)
    same(W.Workload(name, model, W.make_inputs(model, 37, "normal"), muts, ""))


@pytest.mark.parametrize("cfg", ["resnet20", "mobilenetv2"])
def test_chains_in_the_allocation_free_call(cfg):
    wl = W.make_workload(cfg, n_inputs=130, n_mutants=30)
    _, words, kills, score = run_gpu(wl, fused_paths=0)
    import torch
    m = Mure(device=0)
    md = wl.model
    m.load_model(md.nodes, md.in_hwc, md.dtype, md.weights, md.biases)
    m.apply(wl.mutants)
    m.run_original(torch.from_numpy(wl.inputs.view(np.int16)).cuda())
    kb, k2, s2 = m.run_mutants(noalloc=True)
    assert np.array_equal(kb.cpu().numpy().view(np.uint64), words) and np.array_equal(k2, kills) and s2 == score
