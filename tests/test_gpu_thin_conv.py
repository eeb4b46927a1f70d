"""bf16 convolutions of few input channels (conv_thin_kernel): with small
integers every product and sum is exact, so the logits must equal a plain
float32 reference bit for bit -- for the original and for mutants whose changed
channels the gathered-column launch computes."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2607_18582_amd import Mure

pytestmark = pytest.mark.gpu


def bits(x):
    return torch.from_numpy(x.astype(np.float32)).bfloat16().view(torch.int16).numpy().view(np.uint16)


# (H, W, C, C_out, k, stride, pad): one band and several, ragged bands and
# tiles, odd rows, one to eight channels of left padding, 1 to 100 outputs of 16
# and 64 columns; planes on both sides of the size below which the general
# kernel runs; the last two keep the general kernel too (K > 32; W C % 8 != 0)
@pytest.mark.parametrize("shape", [(32, 32, 3, 16, 3, 1, 1), (17, 16, 3, 20, 3, 2, 1), (9, 8, 1, 4, 5, 1, 2),
                                   (12, 8, 2, 64, 4, 2, 0), (40, 24, 3, 100, 3, 1, 0), (5, 8, 4, 24, 2, 1, 2),
                                   (8, 8, 3, 48, 3, 1, 1), (8, 8, 3, 64, 3, 1, 1), (12, 8, 3, 64, 3, 1, 1),
                                   (18, 8, 4, 24, 2, 1, 2), (66, 8, 8, 32, 1, 1, 0), (17, 8, 3, 64, 3, 1, 1),
                                   (1, 1, 32, 512, 1, 1, 0), (33, 1, 8, 32, 1, 1, 0), (16, 16, 4, 16, 3, 1, 1), (10, 10, 3, 16, 3, 1, 1)])
def test_thin_conv_is_exact(shape):
    h, w, c, cout, k, stride, pad = shape
    rng = np.random.default_rng(3)
    b = W.configs._Builder((h, w, c))
    x = b.conv(0, cout, k, stride=stride, pad=pad, relu=True)
    b.dense(x, 3, False)
    ho, wo, _ = b.nodes[x].out_hwc
    wc, bc = rng.integers(-1, 2, (cout, k, k, c)), rng.integers(-3, 4, cout)
    wd, bd = rng.integers(-1, 2, (3, ho * wo * cout)), rng.integers(-3, 4, 3)
    n = 5
    xs = rng.integers(-2, 3, (n, h, w, c))

    def logits(wc, bc):
        y = torch.nn.functional.conv2d(torch.from_numpy(xs).permute(0, 3, 1, 2).float(),
                                       torch.from_numpy(wc).permute(0, 3, 1, 2).float(),
                                       torch.from_numpy(bc).float(), stride, pad).clamp(min=0)
        return (y.permute(0, 2, 3, 1).reshape(n, -1) @ torch.from_numpy(wd).float().T + torch.from_numpy(bd).float()).numpy()

    m = Mure(device=0)
    m.load_model(b.nodes, (h, w, c), "bf16", [None, bits(wc), bits(wd)],
                 [None, bc.astype(np.float32), bd.astype(np.float32)])
    # mutants: fuzz by whole numbers of one neuron, inverse of another, both of a third pair
    noise = rng.integers(-1, 2, (2, k * k * c)).astype(np.float32)
    recs = [(0, W.GF, 0, noise[0]), (1, W.NAI, cout - 1, None), (2, W.GF, cout - 1, noise[1]), (2, W.GF, 1, noise[0])]
    m.apply_mutants(3, [r[0] for r in recs], [r[1] for r in recs], [1] * 4, [r[2] for r in recs], [-1] * 4,
                    [r[3] for r in recs])
    m.run_original(torch.from_numpy(bits(xs).view(np.int16)).cuda())
    assert np.array_equal(m.get_logits(-1).cpu().numpy(), logits(wc, bc))
    for mutant in range(3):
        w2, b2 = wc.copy(), bc.copy()
        for who, op, i, eps in recs:
            if who == mutant and op == W.GF:
                w2[i] += eps.reshape(k, k, c).astype(int)
            elif who == mutant:
                w2[i], b2[i] = -w2[i], -b2[i]
        assert np.array_equal(m.get_logits(mutant).cpu().numpy(), logits(w2, b2)), mutant
