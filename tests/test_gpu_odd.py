"""Odd hidden sizes on the weight-stationary fp32 cell (rows of any alignment; the last request of a row covers up to three
elements of whatever follows it): every scheduler that sums in the common order gives the host-driven scheduler's bits,
and every node agrees with the checker (fp32 sums of at most 1 024 products of order one: 1e-6 each way)."""
import numpy as np
import pytest

import oracle
from paper_1809_00832_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell", ["lstm", "rnn"])
@pytest.mark.parametrize("H", [1, 2, 3, 35, 63, 129, 257, 321, 383, 385, 511])
def test_odd_sizes_give_the_same_bits_everywhere(H, cell):
    print("case odd", cell, H, flush=True)
    if cell == "lstm":
        params = synth.make_treelstm_params(800 + H, 50, 21, H, "xavier")
    else:
        params = synth.make_rnn_params(800 + H, synth.CELL_TREERNN, 50, H, scale=0.5 / H ** 0.5)
    trees = synth.make_trees(801, [1, 2, 30, 1, 7, 65, 3, 18], ["random", "chain"] * 4, 50)
    ref = oracle.forward_params(params, trees, n_threads=8)
    first = None
    for sched in ("level_host", "level_device", "ready", "ready_priority"):
        net = binding.TreeNet(params, scheduler=sched)
        try:
            got = net.run(trees)
            for _ in range(2):
                net.batch["h"].fill_(float("nan"))       # (rows behind a row's end must not matter)
                net.forward()
                assert binding.tl_status(net.ctx) == 0
                assert np.array_equal(net.batch["h"].cpu().numpy(), got["h"])
        finally:
            net.close()
        np.testing.assert_allclose(got["h"], ref["h"], rtol=1e-5, atol=2e-6, err_msg=sched)
        if first is None:
            first = got["h"]
        assert np.array_equal(got["h"], first), sched
