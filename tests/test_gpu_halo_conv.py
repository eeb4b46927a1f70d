"""bf16 3x3 stride-1 convolutions on LDS halo tiles (conv_halo_kernel) at every
width and image height the kernel's pixel layout distinguishes: with small
integers every product and sum is exact, so the logits must equal a plain
float32 reference bit for bit -- whole rows, pooled rows and an identity
shortcut (its two-pass epilogue), and gathered columns of mutants -- in
launches of few blocks (32 columns each) and of more than one per CU (64)."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2607_18582_amd import Mure

pytestmark = pytest.mark.gpu


def bits(x):
    return torch.from_numpy(x.astype(np.float32)).bfloat16().view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("form", ["plain", "pool", "add"])
@pytest.mark.parametrize("h,w,c,cout", [(8, 8, 16, 64), (16, 8, 32, 32), (32, 8, 16, 32), (64, 8, 16, 64),
                                        (16, 16, 48, 32), (32, 16, 16, 64), (16, 32, 16, 96), (48, 32, 32, 32),
                                        (8, 64, 16, 64), (64, 64, 16, 32)])
def test_halo_conv_is_exact(h, w, c, cout, form, many):
    rng = np.random.default_rng(5)
    n = 11 if h * w <= 512 else 3                        # several images a band, a ragged last one
    if many:
        n += 256 * 512 // (h * w)                        # more than 256 bands
    b = W.configs._Builder((h, w, c))
    if form == "add":
        cout = c if c % 32 == 0 else 32
        x0 = b.conv(0, cout, 1, relu=False)              # the shortcut: 1x1, exact
        a = b.conv(x0, cout, 3, pad=1, relu=False)
        x = b.add(a, x0, relu=True)
    else:
        x0 = None
        a = x = b.conv(0, cout, 3, pad=1, relu=True, pool=2 if form == "pool" else 0)
    g = b.gap(x) if form != "pool" else x
    b.dense(g, 3, False)
    ints = lambda *s: rng.integers(-1, 2, s)
    p = {i: (ints(nd.c_out, nd.kh, nd.kw, nd.c_in) if nd.kind == W.CONV2D else ints(nd.c_out, nd.c_in),
             rng.integers(-2, 3, nd.c_out)) for i, nd in enumerate(b.nodes) if nd.kind in (W.CONV2D, W.DENSE)}
    # few non-zero inputs and weights keep every value below 256, exact in bfloat16
    for i in p:
        if b.nodes[i].kind == W.CONV2D:
            p[i] = (p[i][0] * (rng.random(p[i][0].shape) < 12.0 / p[i][0][0].size), p[i][1])
    xs = ints(n, h, w, c) * (rng.random((n, h, w, c)) < 0.5)

    def logits(p):
        conv = lambda y, i: torch.nn.functional.conv2d(y, torch.from_numpy(p[i][0]).permute(0, 3, 1, 2).float(),
                                                       torch.from_numpy(p[i][1]).float(), padding=b.nodes[i].pad)
        y = torch.from_numpy(xs).permute(0, 3, 1, 2).float()
        if x0 is not None:
            y = conv(y, x0)
            assert float(y.abs().max()) <= 256
            y = (conv(y, a) + y).clamp(min=0)
        else:
            y = conv(y, a).clamp(min=0)
        assert float(y.abs().max()) <= 256
        if form == "pool":
            y = torch.nn.functional.max_pool2d(y, 2).permute(0, 2, 3, 1).reshape(n, -1)
        else:
            # the GAP sums exactly and rounds its mean to bfloat16
            y = (y.sum((2, 3)) * np.float32(1.0 / (h * w))).bfloat16().float()
        d = len(b.nodes) - 1
        return (y.double() @ torch.from_numpy(p[d][0]).double().T + torch.from_numpy(p[d][1]).double()).float().numpy()

    m = Mure(device=0)
    m.load_model(b.nodes, (h, w, c), "bf16", [bits(p[i][0]) if i in p else None for i in range(len(b.nodes))],
                 [p[i][1].astype(np.float32) if i in p else None for i in range(len(b.nodes))])
    recs = [(0, W.NAI, 0, -1), (1, W.NEB, cout - 1, -1), (2, W.NS, 1, cout - 2), (2, W.NAI, cout // 2, -1)]
    m.apply_mutants(3, [r[0] for r in recs], [r[1] for r in recs], [a] * 4, [r[2] for r in recs],
                    [r[3] for r in recs], [None] * 4)
    m.run_original(torch.from_numpy(bits(xs).view(np.int16)).cuda())
    tol = dict(rtol=0, atol=0) if form == "pool" else dict(rtol=2e-6, atol=1e-6)   # a mean's float32 dot product
    np.testing.assert_allclose(m.get_logits(-1).cpu().numpy(), logits(p), **tol)
    for mutant in range(3):
        q = dict(p)
        w2, b2 = p[a][0].copy(), p[a][1].copy()
        for who, op, i, j in recs:
            if who != mutant:
                continue
            if op == W.NAI:
                w2[i], b2[i] = -w2[i], -b2[i]
            elif op == W.NEB:
                w2[i], b2[i] = 0, 0
            else:
                w2[[i, j]], b2[[i, j]] = w2[[j, i]], b2[[j, i]]
        q[a] = (w2, b2)
        np.testing.assert_allclose(m.get_logits(mutant).cpu().numpy(), logits(q), **tol, err_msg=str(mutant))
