"""The wide LSTM kernel with 64 and with 16 rows per block gives the same
values: a run of many mutants takes the one, a single mutant's logits the
other (lstm_wide_rows)."""
import numpy as np
import pytest

import workloads as W
from harness import device_inputs, run_gpu, sample_mutants, unpack_words
from paper_2607_18582_amd import Mure

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1000, 961])               # whole blocks of 16 and 64 rows; one row past both
def test_lstm_rows_per_block(n):
    wl = W.make_workload("rnn_imdb", n_inputs=n, n_mutants=300)
    m, words, kills, score = run_gpu(wl)
    kill = unpack_words(words, n)
    label = m.get_logits(-1).cpu().numpy().argmax(1)
    for mid in sample_mutants(m, wl):
        assert np.array_equal(m.get_logits(mid).cpu().numpy().argmax(1) != label, kill[mid]), mid


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
