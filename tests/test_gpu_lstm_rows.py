"""The wide LSTM kernel with 64 and with 16 rows per block gives the same
logits, bit for bit: a launch over 16,384 inputs of one model takes the one, a
launch over about 1,000 the other (lstm_wide_rows)."""
import numpy as np
import pytest

import workloads as W
from harness import device_inputs, run_gpu, sample_mutants, unpack_words
from paper_2607_18582_amd import Mure

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1024, 961])               # whole blocks of 16 and 64 rows; one row past both
def test_lstm_rows_per_block(n):
    wl = W.make_workload("rnn_imdb", n_inputs=n, n_mutants=300)
    m, words, kills, score = run_gpu(wl)                 # many slots: 64 rows
    kill = unpack_words(words, n)
    mids = [-1] + sample_mutants(m, wl)
    small = [m.get_logits(mid).cpu().numpy() for mid in mids]
    x = device_inputs(wl)
    m.run_original(x.repeat([16384 // n + 1] + [1] * (x.dim() - 1))[:16384].contiguous())
    for mid, z in zip(mids, small):
        big = m.get_logits(mid).cpu().numpy()
        for i in range(0, 16384, n):
            assert np.array_equal(big[i:i + n], z[:16384 - i]), (mid, i)
        if mid >= 0:
            assert np.array_equal(z.argmax(1) != small[0].argmax(1), kill[mid]), mid


@pytest.mark.parametrize("cfg", ["rnn_imdb", "lstm"])      # the wide kernel and the LDS kernel
@pytest.mark.parametrize("value,finite", [(np.nan, False), (-3e38, True), (3e38, True)])
def test_lstm_gates_saturate_and_pass_nan(cfg, value, finite):
    """A gate of +-infinity (or nearly) is 1 or 0; a NaN reaches the logits."""
    wl = W.make_workload(cfg, n_inputs=70, n_mutants=3)
    md = wl.model
    lstm = [i for i, n in enumerate(md.nodes) if n.kind == W.LSTM][0]
    node = md.nodes[lstm]
    w = [None if x is None else x.copy() for x in md.weights]
    w[lstm].reshape(node.c_out, 4, -1)[5, 1, -1] = value   # a forget gate's bias
    m = Mure(device=0)
    m.load_model(md.nodes, md.in_hwc, md.dtype, w, md.biases)
    m.apply(wl.mutants)
    m.run_original(device_inputs(wl))
    z = m.get_logits(-1).cpu().numpy()
    assert np.isfinite(z).all() == finite and (finite or np.isnan(z).all())
    _, _, score = m.run_mutants()
    assert (score["nonfinite_logits"] == 0) == finite
