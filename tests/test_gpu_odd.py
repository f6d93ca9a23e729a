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


@pytest.mark.parametrize("cell", ["lstm", "rnn"])
@pytest.mark.parametrize("H", [5, 18, 23, 30, 31])
def test_rows_of_one_k_step(H, cell):
    """Up to H = 32 the elements of a request are asked for one by one, those behind the row's end beyond the table."""
    test_odd_sizes_give_the_same_bits_everywhere(H, cell)


@pytest.mark.parametrize("cell,H", [("lstm", h) for h in (1, 3, 16, 25, 26, 51, 77, 150, 205, 308, 359, 411, 461, 510)] +
                         [("rnn", h) for h in (1, 50, 127, 129, 255, 301, 450)])
def test_backward_in_one_kernel_at_any_size(cell, H):
    """The weight-stationary operand gradient pads rows of gate gradients to a multiple of 128 values; what lies behind a row's end
    does not matter: the gradients that reach the leaves are those of the launches per height bit for bit, and agree with
    the checker (sums of at most 2 600 products of order one)."""
    import torch
    print("case backward sizes", cell, H, flush=True)
    if cell == "lstm":
        params = synth.make_treelstm_params(820 + H, 50, 21, H, "xavier")
    else:
        params = synth.make_rnn_params(820 + H, synth.CELL_TREERNN, 50, H, scale=0.5 / H ** 0.5)
    trees = synth.make_trees(821, [1, 2, 30, 1, 7, 65, 3, 18], ["random", "chain"] * 4, 50)
    g_h = torch.from_numpy(np.random.default_rng(H).standard_normal((trees.n_nodes, H)).astype(np.float32)).cuda()
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        b = net.load(trees)
        binding.tl_set_keep_gates(net.ctx, True)
        net.forward()
        out = {}
        for mode in (-1, 0, 1):
            binding.tl_set_async_backward(net.ctx, mode)
            out[mode] = {k: v.cpu().numpy() for k, v in binding.tl_backward(net.ctx, b, g_h, params.embed_dim).items()}
            assert binding.tl_status(net.ctx) == 0
        h, c = b["h"].cpu().numpy(), b["c"].cpu().numpy() if b["c"] is not None else None
    finally:
        net.close()
    ref = oracle.backward(params, trees, h, c, g_h.cpu().numpy())
    for mode in (0, 1):
        assert np.array_equal(out[mode]["d_x"], out[-1]["d_x"]), mode
    for k in ref:
        np.testing.assert_allclose(out[0][k], ref[k], rtol=1e-4, atol=1e-4 * max(1.0, float(np.abs(ref[k]).max())), err_msg=k)


@pytest.mark.parametrize("H,n_trees,leaves,shape", [(500, 40, 50, "random"), (500, 42, 50, "random"), (500, 7, 300, "chain"), (340, 40, 98, "random"), (340, 42, 98, "random"),
                                                    (340, 14, 300, "chain")])
def test_backward_of_many_nodes_on_both_sides_of_the_lines(H, n_trees, leaves, shape):
    """Sizes whose batches of many nodes take launches per height by default (2 000 internal nodes at H = 500, 4 000 at H = 340), deep
    trees or calls that do not wait one kernel or the other: the same bits of d_x in every mode."""
    import torch
    print("case backward lines", H, n_trees, leaves, shape, flush=True)
    params = synth.make_treelstm_params(830 + H, 50, 21, H, "xavier")
    trees = synth.make_trees(831, [leaves + t % 3 for t in range(n_trees)], [shape] * n_trees, 50)
    g_h = torch.from_numpy(np.random.default_rng(H).standard_normal((trees.n_nodes, H)).astype(np.float32)).cuda()
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        b = net.load(trees)
        binding.tl_set_keep_gates(net.ctx, True)
        net.forward()
        out = {}
        for mode in (-1, 0, 1):
            binding.tl_set_async_backward(net.ctx, mode)
            out[mode] = {k: v.cpu().numpy() for k, v in binding.tl_backward(net.ctx, b, g_h, params.embed_dim).items()}
            assert binding.tl_status(net.ctx) == 0
    finally:
        net.close()
    assert np.abs(out[-1]["d_x"]).max() > 0
    for mode in (0, 1):
        assert np.array_equal(out[mode]["d_x"], out[-1]["d_x"]), mode
        for k in out[mode]:
            np.testing.assert_allclose(out[mode][k], out[-1][k], rtol=1e-4, atol=2e-5 * float(np.abs(out[-1][k]).max()), err_msg=k)
