"""The backward pass that mirrors the data-flow forward (csrc/back_flow.hpp: TreeLSTM from kept activations and TreeRNN at H <= 512), at the
edges of its layout, against the CPU checker and in all modes of tl_set_async_backward, whose gradients of the leaves must agree bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1809_00832_amd import binding, synth

pytestmark = pytest.mark.gpu


def make(cell, H, seed, counts, shapes, E=21):
    if cell == "lstm":
        params = synth.make_treelstm_params(seed, 50, E, H, "xavier")
    else:
        params = synth.make_rnn_params(seed, synth.CELL_TREERNN, 50, H, scale=0.5 / H ** 0.5)
    return params, synth.make_trees(seed + 1, counts, shapes, 50)


def backward(params, trees, g_h, modes=(0,), keep=True):
    """{mode: gradients} and the states of one forward."""
    net = binding.TreeNet(params, scheduler="dataflow")
    out = {}
    try:
        b = net.load(trees)
        binding.tl_set_keep_gates(net.ctx, keep)
        net.forward()
        g = torch.from_numpy(g_h).cuda()
        for mode in modes:
            binding.tl_set_async_backward(net.ctx, mode)
            out[mode] = {k: v.cpu().numpy() for k, v in binding.tl_backward(net.ctx, b, g, params.embed_dim).items()}
            assert binding.tl_status(net.ctx) == 0
        h = b["h"].cpu().numpy()
        c = b["c"].cpu().numpy() if b["c"] is not None else None
    finally:
        net.close()
    return out, h, c


# H: one unit, one and two column groups, an odd number of them, whole and ragged pairs, the largest of each number of pairs per wave and the size behind it;
# E: leaves' columns in one group of three and beyond
@pytest.mark.parametrize("cell,H,E", [("lstm", h, e) for h, e in ((2, 1), (17, 16), (32, 48), (33, 49), (48, 300), (128, 300), (129, 21), (256, 257), (257, 64), (384, 96), (385, 7), (512, 97))] +
                         [("rnn", h, h) for h in (2, 31, 33, 128, 130, 257, 512)])
def test_sizes_at_the_edges_of_the_layout(cell, H, E):
    print("case back sizes", cell, H, E, flush=True)
    params, trees = make(cell, H, 900 + H, [1, 2, 40, 1, 9, 70, 3, 18, 33], ["random", "chain", "balanced"] * 3, E)
    g_h = np.random.default_rng(H).standard_normal((trees.n_nodes, H)).astype(np.float32)
    out, h, c = backward(params, trees, g_h, (-1, 0, 1))
    for mode in (0, 1):
        assert np.array_equal(out[mode]["d_x"], out[-1]["d_x"]), mode
    ref = oracle.backward(params, trees, h, c, g_h)
    for k in ref:                                             # sums of at most 2 600 products of order one (fp32: 2600 * 2^-24 = 1.5e-4 of the largest at worst)
        np.testing.assert_allclose(out[0][k], ref[k], rtol=1e-4, atol=1e-4 * max(1.0, float(np.abs(ref[k]).max())), err_msg=k)


@pytest.mark.parametrize("cell,H", [("lstm", 40), ("lstm", 150), ("rnn", 64)])
@pytest.mark.parametrize("shape", ["balanced", "chain"])
def test_few_large_trees_of_either_kind(cell, H, shape):
    """Fewer trees than sets of workgroups, 256 nodes a tree and more: bushy trees are walked height by height by all workgroups, narrow ones stay with one
    set each; the device picks."""
    print("case back few large", cell, H, shape, flush=True)
    params, trees = make(cell, H, 950 + H, [300, 301, 290], [shape] * 3)
    g_h = np.random.default_rng(H).standard_normal((trees.n_nodes, H)).astype(np.float32)
    out, h, c = backward(params, trees, g_h, (-1, 0, 1, 0))
    for mode in (0, 1):
        assert np.array_equal(out[mode]["d_x"], out[-1]["d_x"]), mode
    ref = oracle.backward(params, trees, h, c, g_h)
    for k in ref:
        np.testing.assert_allclose(out[0][k], ref[k], rtol=1e-4, atol=1e-4 * max(1.0, float(np.abs(ref[k]).max())), err_msg=k)


@pytest.mark.parametrize("cell,H", [("lstm", 150), ("rnn", 100)])
def test_gradients_of_any_size(cell, H):
    """A row of gate gradients is scaled by itself, and so are its pieces of 16 units: trees whose upstream gradients are 2^-60 ... 2^60 times those of others, and within
    one tree units 16 ... 31 2^12 times the others.  d_x of every tree against the checker, relative to the tree's largest value (an operand is met to 2^-22 of its
    piece's largest value, a product to 2^-21: sums of some hundred of them, over at most 12 heights, to 1e-4)."""
    print("case back scales", cell, H, flush=True)
    params, trees = make(cell, H, 970, [30] * 13, ["random"] * 13)
    rng = np.random.default_rng(5)
    g_h = rng.standard_normal((trees.n_nodes, H))
    off = trees.tree_off
    for t in range(12):
        g_h[off[t]:off[t + 1]] *= 2.0 ** (10 * t - 60)
    g_h[off[12]:, 16:32] *= 2.0 ** 12
    g_h = g_h.astype(np.float32)
    out, h, c = backward(params, trees, g_h)
    ref = oracle.backward(params, trees, h, c, g_h)["d_x"]
    for t in range(13):
        rows = slice(off[t], off[t + 1])
        err, top = np.abs(out[0]["d_x"][rows] - ref[rows]).max(), np.abs(ref[rows]).max()
        assert top > 0 and err <= 1e-4 * top, (t, err / top)


@pytest.mark.parametrize("bits", [0x7F800000, 0xFF800000, 0x7FC00000, 0xFFFFFFFF])
@pytest.mark.parametrize("H", [40, 150])
def test_infinities_and_nans_upstream(H, bits):
    """An upstream infinity or NaN - the NaN of 32 ones, which marks rows that are not written yet, among them - comes out as the checker's, and the call ends; trees without one are
    as they were."""
    print("case back non-finite", H, hex(bits), flush=True)
    params, trees = make("lstm", H, 990, [20, 21, 22, 1], ["random", "chain", "random", "random"])
    g_h = np.random.default_rng(7).standard_normal((trees.n_nodes, H)).astype(np.float32)
    clean, _, _ = backward(params, trees, g_h)
    bad = g_h.copy()
    node = int(trees.tree_off[1]) + 3                         # below the root of the chain
    bad.view(np.uint32)[node, 17] = bits
    out, h, c = backward(params, trees, bad, (-1, 0, 1))
    ref = oracle.backward(params, trees, h, c, bad)["d_x"]
    hit = slice(trees.tree_off[1], trees.tree_off[2])
    for mode in (-1, 0, 1):
        got = out[mode]["d_x"]
        assert np.array_equal(np.isfinite(got[hit]), np.isfinite(ref[hit])), mode
        assert not np.isfinite(got[hit]).all()
        mask = np.ones(trees.n_nodes, bool)
        mask[hit] = False
        assert np.array_equal(got[mask], clean[0]["d_x"][mask]), mode


@pytest.mark.parametrize("cell,H", [("lstm", 72), ("rnn", 96)])
@pytest.mark.parametrize("keep", [True, False])
def test_backward_after_an_update_is_that_of_a_fresh_context(cell, H, keep):
    """tl_sgd_update rebuilds the packed transposed matrices (those of the other forms when they are next used)."""
    print("case back update", cell, H, keep, flush=True)
    params, trees = make(cell, H, 1010, [12, 30, 1, 7], ["random"] * 4)
    g_h = np.random.default_rng(9).standard_normal((trees.n_nodes, H)).astype(np.float32)
    g = torch.from_numpy(g_h).cuda()
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        b = net.load(trees)
        binding.tl_set_keep_gates(net.ctx, keep)
        for _ in range(2):
            net.forward()
            grads = binding.tl_backward(net.ctx, b, g, params.embed_dim)
            binding.tl_sgd_update(net.ctx, 0.05, b, grads)
        net.forward()
        after = binding.tl_backward(net.ctx, b, g, params.embed_dim)["d_x"].cpu().numpy()
        new = {k: v.cpu().numpy() for k, v in binding.tl_get_params(net.ctx, params.vocab, params.embed_dim, params.hidden, params.cell).items()}
    finally:
        net.close()
    q = synth.Params(params.cell, params.vocab, params.embed_dim, params.hidden, new["emb"], new.get("w_leaf"), new.get("b_leaf"), new["u"], new["b"], None)
    fresh, _, _ = backward(q, trees, g_h, keep=keep)
    assert np.array_equal(fresh[0]["d_x"], after)


# (H, E, trees of 20 leaves): both products in one launch of the 64 x 64 form with and without 16-byte loads, apart in that form (only one has them), just below and above the
# line from which one launch of the wide form fills the chip (slices of 64 nodes times 30 tiles: from 9 on), and well above with ragged tiles of either matrix
@pytest.mark.parametrize("H,E,n_trees", [(40, 24, 3), (41, 23, 3), (40, 23, 3), (150, 300, 26), (150, 300, 28), (131, 129, 60), (200, 31, 60)])
def test_weight_gradients_of_both_matrices(H, E, n_trees):
    print("case both weight gradients", H, E, n_trees, flush=True)
    params, trees = make("lstm", H, 700 + H + n_trees, [20] * n_trees, ["random"] * n_trees, E)
    g_h = np.random.default_rng(H).standard_normal((trees.n_nodes, H)).astype(np.float32)
    for keep in (True, False):                                # (rows of gate gradients by node, and by list position)
        out, h, c = backward(params, trees, g_h, keep=keep)
        ref = oracle.backward(params, trees, h, c, g_h)
        for k in ref:                                         # sums of at most 1 200 products, fp32: 1200 * 2^-24 = 7e-5 of the largest at worst
            np.testing.assert_allclose(out[0][k], ref[k], rtol=1e-4, atol=1e-4 * max(1.0, float(np.abs(ref[k]).max())), err_msg=k)


def replayed(step):
    """A graph of `step`, recorded on a stream of its own; what step returned in it."""
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        out = step()
    return graph, out


def params_of(net, params):
    new = {k: v.cpu().numpy() for k, v in binding.tl_get_params(net.ctx, params.vocab, params.embed_dim, params.hidden, params.cell).items()}
    rntn = params.cell == synth.CELL_RNTN
    return synth.Params(params.cell, params.vocab, params.embed_dim, params.hidden, new["emb"], None if rntn else new.get("w_leaf"), new.get("b_leaf"), new["u"], new["b"],
                        new["w_leaf"] if rntn else None)


def test_replayed_training_step():
    """Forward, backward (which does not wait) and update as one graph: three replays, eager work between them, are three eager steps."""
    print("case back replayed step", flush=True)
    params, trees = make("lstm", 72, 1100, [12, 30, 1, 7], ["random"] * 4)
    g = torch.from_numpy(np.random.default_rng(3).standard_normal((trees.n_nodes, 72)).astype(np.float32)).cuda()
    states = []
    for graphed in (False, True):
        net = binding.TreeNet(params, scheduler="dataflow")
        try:
            b = net.load(trees)
            binding.tl_set_keep_gates(net.ctx, True)
            binding.tl_set_async_backward(net.ctx, 1)

            def step():
                net.forward()
                grads = binding.tl_backward(net.ctx, b, g, params.embed_dim)
                binding.tl_sgd_update(net.ctx, 0.05, b, grads)
                return grads
            step()                                            # eager: sizes the workspaces
            torch.cuda.synchronize()
            if graphed:
                graph, grads = replayed(step)
            for _ in range(3):
                if graphed:
                    graph.replay()
                else:
                    grads = step()
                torch.cuda.synchronize()
                assert torch.isfinite(torch.randn(1 << 16, device="cuda").sum())
            assert binding.tl_status(net.ctx) == 0
            states.append((grads["d_x"].cpu().numpy(), params_of(net, params)))
        finally:
            net.close()
    (dx0, p0), (dx1, p1) = states
    top = np.abs(dx0).max()
    assert np.abs(dx1 - dx0).max() <= 1e-5 * top              # (embedding rows and weight gradients are summed with atomics: last bits)
    assert np.abs(p1.u - p0.u).max() <= 1e-5 * np.abs(p0.u).max() and np.abs(p0.u - params.u).max() > 1e-3


@pytest.mark.parametrize("cell", ["lstm", "rntn"])
def test_eager_backward_after_replayed_updates(cell):
    """A replay changes the parameters without a call: matrices that an update does not rebuild itself, packed by an eager backward pass before, are packed again.
    (TreeLSTM: gates recomputed; RNTN: launches per height.)"""
    print("case back after replayed updates", cell, flush=True)
    H = 48
    if cell == "lstm":
        params, trees = make("lstm", H, 1110, [12, 30, 1, 7], ["random"] * 4)
    else:
        params = synth.make_rnn_params(1110, synth.CELL_RNTN, 50, H, scale=0.3 / H)
        trees = synth.make_trees(1111, [12, 30, 1, 7], ["random"] * 4, 50)
    rntn = cell == "rntn"
    g = torch.from_numpy(np.random.default_rng(4).standard_normal((trees.n_nodes, H)).astype(np.float32)).cuda()

    def gradients(net):
        net.forward()
        return binding.tl_backward(net.ctx, net.batch, g, params.embed_dim, rntn=rntn)
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        b = net.load(trees)
        binding.tl_set_async_backward(net.ctx, -1)
        grads = gradients(net)
        torch.cuda.synchronize()
        graph, _ = replayed(lambda: binding.tl_sgd_update(net.ctx, 0.05, b, grads))
        for _ in range(2):
            gradients(net)                                    # packs them
            graph.replay()
            torch.cuda.synchronize()
            after = gradients(net)["d_x"].cpu().numpy()
            q = params_of(net, params)
            assert np.abs(q.u - params.u).max() > 1e-3
            fresh = binding.TreeNet(q, scheduler="dataflow")
            try:
                fresh.load(trees)
                binding.tl_set_async_backward(fresh.ctx, -1)
                want = gradients(fresh)["d_x"].cpu().numpy()
            finally:
                fresh.close()
            assert np.array_equal(after, want)
    finally:
        net.close()


def test_replayed_backward_of_a_batch_beyond_the_tables():
    """A batch whose rows need more than 32-bit offsets takes the fp32 matrices: a recorded backward pass packs them, whatever was packed when it was recorded."""
    H, E = 512, 16
    params, trees = make("lstm", H, 1120, [4096] * 52, ["balanced"] * 52, E)
    assert trees.n_nodes * H * 20 >= 1 << 32
    print("case back beyond the tables", trees.n_nodes, flush=True)
    torch.manual_seed(5)
    g = torch.randn((trees.n_nodes, H), device="cuda")

    def prepared(p):
        net = binding.TreeNet(p, scheduler="dataflow")
        b = net.load(trees)
        binding.tl_set_keep_gates(net.ctx, True)
        binding.tl_set_async_backward(net.ctx, 1)
        return net, b

    def gradients(net, b):
        net.forward()
        return binding.tl_backward(net.ctx, b, g, E)
    net, b = prepared(params)
    try:
        grads = gradients(net, b)
        torch.cuda.synchronize()
        graph, recorded = replayed(lambda: gradients(net, b))
        step = 0.02 / float(grads["d_u"].abs().max())
        for _ in range(2):
            binding.tl_sgd_update(net.ctx, step, b, grads, with_embedding=False)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
        assert binding.tl_status(net.ctx) == 0
        q = params_of(net, params)
    finally:
        net.close()
    assert np.abs(q.u - params.u).max() > 1e-2
    fresh, b = prepared(q)
    try:
        want = gradients(fresh, b)
        assert binding.tl_status(fresh.ctx) == 0
        assert torch.equal(recorded["d_x"], want["d_x"])
    finally:
        fresh.close()


def test_rows_beyond_two_gib():
    """The copy that the blocks read may be of nearly 4 GiB: offsets of its upper half (TreeLSTM, H = 2: 640 bytes a row, 3.5 million internal nodes).
    The same tree over and over: every copy's d_x has the bits of a batch of two."""
    L, n_trees, H, E = 64, 56000, 2, 3
    params, two = make("lstm", H, 1130, [L] * 2, ["random"] * 2, E)
    n = int(two.tree_off[1])
    one = [a[:n] for a in (two.left, two.right, two.word)]

    def repeated(count):
        base = (np.arange(count, dtype=np.int32) * n)[:, None]
        child = lambda a: np.where(a >= 0, a + base, -1).astype(np.int32).ravel()
        return synth.TreeBatch((np.arange(count + 1) * n).astype(np.int32), child(one[0]), child(one[1]), np.tile(one[2], count))
    g = np.random.default_rng(11).standard_normal((n, H)).astype(np.float32)
    got = {}
    for count in (2, n_trees):
        trees = repeated(count)
        print("case back beyond 2 GiB", trees.n_nodes, flush=True)
        net = binding.TreeNet(params, scheduler="dataflow")
        try:
            b = net.load(trees)
            binding.tl_set_keep_gates(net.ctx, True)
            net.forward()
            got[count] = binding.tl_backward(net.ctx, b, torch.from_numpy(g).cuda().repeat(count, 1), E)["d_x"].view(count, n, E)
            assert binding.tl_status(net.ctx) == 0
        finally:
            net.close()
    assert (n_trees * (L - 1)) * 640 > 1 << 31
    assert bool((got[n_trees] == got[2][0]).all()) and bool((got[2][1] == got[2][0]).all())


@pytest.mark.parametrize("cell,H", [("lstm", 150), ("lstm", 512), ("rnn", 512)])
def test_a_diverged_step_is_not_slow(cell, H):
    """Sums that are not finite are taken again, one by one; those of a row that holds a NaN are not, they would stay NaN.  Time of a backward pass whose upstream gradients
    are all NaN against that of ordinary ones (taken again throughout: some hundred times as long; the weight gradients' share of it is below twice the whole)."""
    print("case back diverged", cell, H, flush=True)
    params, trees = make(cell, H, 1140, [20] * 60, ["random"] * 60, 200)
    clean = torch.from_numpy(np.random.default_rng(13).standard_normal((trees.n_nodes, H)).astype(np.float32)).cuda()
    net = binding.TreeNet(params, scheduler="dataflow")
    us = []
    try:
        b = net.load(trees)
        binding.tl_set_keep_gates(net.ctx, True)
        for g in (clean, torch.full_like(clean, float("nan"))):
            times = []
            for _ in range(8):
                net.forward()
                begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                begin.record()
                d_x = binding.tl_backward(net.ctx, b, g, params.embed_dim)["d_x"]
                end.record()
                torch.cuda.synchronize()
                times.append(begin.elapsed_time(end) * 1e3)
            us.append(sorted(times)[4])
        leaf = torch.from_numpy(trees.left < 0).cuda()
        assert bool(torch.isnan(d_x[leaf]).all())
    finally:
        net.close()
    assert us[1] < 4 * us[0] + 200, us


@pytest.mark.parametrize("cell,H", [("lstm", h) for h in (96, 150, 300, 512)] + [("rnn", h) for h in (31, 130, 512)])
def test_pieces_far_apart(cell, H):
    """A block-diagonal U (16 units a block, as many as share a power of two) keeps the units' groups apart, and each group's upstream gradients have a size of their own, up to
    2^50 apart: a group's gradients are met to a share of its own largest value, beside larger groups in the same quarter of a row too.  TreeLSTM: d_u and d_b (d_x mixes
    the groups of a quarter of a row, which share a scale there); TreeRNN: d_x.  Tolerance as for gradients of any size."""
    print("case back pieces far apart", cell, H, flush=True)
    params, trees = make(cell, H, 1150, [20, 31, 2, 1], ["random"] * 4)
    group = np.arange(H) // 16
    ng = 5 if cell == "lstm" else 1
    same = np.tile(group[:, None] == group[None, :], (2, ng))
    params.u = np.where(same, params.u * 3, 0).astype(np.float32)
    size = 2.0 ** -np.array([0, 13, 14, 15, 16, 25, 31, 50])[group % 8]
    g_h = (np.random.default_rng(17).standard_normal((trees.n_nodes, H)) * size).astype(np.float32)
    out, h, c = backward(params, trees, g_h, (-1, 0, 1))
    ref = oracle.backward(params, trees, h, c, g_h)
    for mode in (-1, 0, 1):
        for q in range(group[-1] + 1):
            units = np.flatnonzero(group == q)
            if cell == "lstm":
                cols = (np.arange(ng)[:, None] * H + units).ravel()
                pairs = [(out[mode]["d_b"][cols], ref["d_b"][cols]), (out[mode]["d_u"][:, cols], ref["d_u"][:, cols])]
            else:
                pairs = [(out[mode]["d_x"][:, units], ref["d_x"][:, units])]
            for got, want in pairs:
                top = np.abs(want).max()
                assert top > 0 and np.abs(got - want).max() <= 1e-4 * top, (mode, q, np.abs(got - want).max() / top)


@pytest.mark.parametrize("H", [40, 150, 512])
@pytest.mark.parametrize("where", ["u", "w_leaf"])
def test_infinite_weights(where, H):
    """A column with an infinity has no two terms: its sums are taken in fp32 and are finite, infinite or NaN where the oracle's are.  (The infinity is an output gate's, whose
    sigmoid is 0 or 1, so that the states stay finite.)"""
    print("case back infinite weights", where, H, flush=True)
    params, trees = make("lstm", H, 1160, [20, 31, 2, 1], ["random"] * 4)
    if where == "u":
        params.u = params.u.copy()
        params.u[H + 3, 3 * H + 7] = np.inf
    else:
        params.w_leaf = params.w_leaf.copy()
        params.w_leaf[5, H + 9] = np.inf
    g_h = np.random.default_rng(19).standard_normal((trees.n_nodes, H)).astype(np.float32)
    out, h, c = backward(params, trees, g_h, (-1, 0, 1))
    assert np.isfinite(h).all() and np.isfinite(c).all()
    ref = oracle.backward(params, trees, h, c, g_h)["d_x"]
    assert not np.isfinite(ref).all() and (where == "u" or np.isfinite(ref).any())
    for mode in (-1, 0, 1):
        got = out[mode]["d_x"]
        assert np.array_equal(np.isfinite(got), np.isfinite(ref)), mode
        good = np.isfinite(ref)
        np.testing.assert_allclose(got[good], ref[good], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("cell,H", [("rnn", 48), ("rnn", 300), ("lstm", 48), ("lstm", 512)])
def test_sums_that_overflow_only_when_scaled(cell, H):
    """Gradients of 2^120 against weights of 2^-60: the sums are of order 2^60, the scaled ones beyond fp32, and taken again.  TreeRNN: U (only the roots have an upstream
    gradient, so that a leaf's d_x is such a sum or a sum of such); TreeLSTM: W_leaf."""
    print("case back scaled overflow", cell, H, flush=True)
    params, trees = make(cell, H, 1170, [2, 3, 2, 1], ["random"] * 4)
    tiny = np.float32(2.0 ** -60)
    if cell == "rnn":
        params.u = (params.u * tiny).astype(np.float32)
    else:
        params.w_leaf = (params.w_leaf * tiny).astype(np.float32)
    g_h = np.zeros((trees.n_nodes, H))
    roots = np.setdiff1d(np.arange(trees.n_nodes), np.concatenate([trees.left, trees.right]))
    rows = roots if cell == "rnn" else np.flatnonzero(trees.left < 0)
    g_h[rows] = np.random.default_rng(23).standard_normal((len(rows), H)) * 2.0 ** 120
    g_h = g_h.astype(np.float32)
    out, h, c = backward(params, trees, g_h, (-1, 0, 1))
    ref = oracle.backward(params, trees, h, c, g_h)["d_x"]
    for mode in (-1, 0, 1):
        for n in np.flatnonzero(trees.left < 0):
            top = np.abs(ref[n]).max()
            assert 0 < top < 2.0 ** 127 and np.abs(out[mode]["d_x"][n] - ref[n]).max() <= 1e-4 * top, (mode, n)


def one_large_tree(leaves, shape, at, n_small=60, seed=1200):
    """Small trees around one that is large beside them."""
    counts, shapes = [3 + 5 * i % 37 for i in range(n_small)], ["random"] * n_small
    counts.insert(at, leaves)
    shapes.insert(at, shape)
    return synth.make_trees(seed, counts, shapes, 50)


# bushy (all workgroups walk the heights together) and not, first, last and in between; just below and from the line of 1 536 nodes on (a tree of 768 leaves has 1 535; TreeRNN: 1 792)
@pytest.mark.parametrize("cell,H", [("lstm", 20), ("lstm", 150), ("lstm", 512), ("rnn", 64), ("rnn", 130), ("rnn", 512)])
@pytest.mark.parametrize("leaves,shape,at", [(768, "random", 30), (769, "random", 30), (2500, "random", 0), (2500, "balanced", 60), (1500, "chain", 7)])
def test_a_tree_that_is_large_beside_the_others(cell, H, leaves, shape, at):
    print("case back skewed", cell, H, leaves, shape, flush=True)
    params, _ = make(cell, H, 1200 + H, [1], ["random"])
    if cell == "rnn" and leaves < 1000:
        leaves += 128
    trees = one_large_tree(leaves, shape, at)
    g_h = np.random.default_rng(H).standard_normal((trees.n_nodes, H)).astype(np.float32)
    out, h, c = backward(params, trees, g_h, (-1, 0, 1, 0))
    for mode in (0, 1):
        assert np.array_equal(out[mode]["d_x"], out[-1]["d_x"]), mode
    ref = oracle.backward(params, trees, h, c, g_h)
    for k in ref:                                             # sums of at most 3 700 products, fp32, by slices of the nodes: as in the tests above
        np.testing.assert_allclose(out[0][k], ref[k], rtol=1e-4, atol=1e-4 * max(1.0, float(np.abs(ref[k]).max())), err_msg=k)


def test_a_large_tree_in_a_replayed_step():
    """The same in a graph: what the kernels count for their choice starts from zero in every replay, for a batch of either kind."""
    H = 64
    params, _ = make("lstm", H, 1250, [1], ["random"])
    for shape in ("random", "chain"):
        print("case back skewed replayed", shape, flush=True)
        trees = one_large_tree(1000, shape, 11)
        g = torch.from_numpy(np.random.default_rng(3).standard_normal((trees.n_nodes, H)).astype(np.float32)).cuda()
        net = binding.TreeNet(params, scheduler="dataflow")
        try:
            b = net.load(trees)
            binding.tl_set_keep_gates(net.ctx, True)
            binding.tl_set_async_backward(net.ctx, 1)

            def step():
                net.forward()
                return binding.tl_backward(net.ctx, b, g, params.embed_dim)
            want = step()["d_x"].clone()
            torch.cuda.synchronize()
            graph, got = replayed(step)
            for _ in range(3):
                got["d_x"].fill_(float("nan"))
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(got["d_x"], want)
                assert torch.isfinite(torch.randn(1 << 16, device="cuda").sum())
            assert binding.tl_status(net.ctx) == 0
        finally:
            net.close()


@pytest.mark.parametrize("what", ["cycle", "roots", "root of the large tree"])
@pytest.mark.parametrize("cell", ["lstm", "rnn"])
@pytest.mark.parametrize("mode", [0, 1, -1])
def test_malformed_batches_with_a_large_tree(cell, what, mode):
    """Where the heights are walked, the walk's own preparation finds what the schedule finds elsewhere: nodes that no leaf leads to, a tree of two roots and one of none.
    The context goes on."""
    print("case back skewed malformed", cell, what, mode, flush=True)
    H = 40
    params, _ = make(cell, H, 1260, [1], ["random"])
    good = one_large_tree(1000, "random", 20, seed=1261)
    ranges = [tuple(np.where(a[lo:hi] >= 0, a[lo:hi] - s, -1) for a, s in ((good.left, lo), (good.right, lo), (good.word, 0))) for lo, hi in zip(good.tree_off[:-1], good.tree_off[1:])]
    word = lambda l: np.where(l < 0, 3, -1)
    if what == "cycle":                                       # a tree of three nodes beside a ring of two with two leaves
        l, r = np.array([1, -1, -1, 4, 3, -1, -1]), np.array([2, -1, -1, 5, 6, -1, -1])
        ranges.insert(40, (l, r, word(l)))
    else:                                                     # two roots; a ring without one
        if what == "roots":
            l, r = np.array([1, -1, -1, 4, -1, -1]), np.array([2, -1, -1, 5, -1, -1])
            ranges.insert(5, (l, r, word(l)))
        else:                                                 # the large tree and a small one in one range
            a, b = ranges[20], ranges[21]
            n = len(a[0])
            ranges[20:22] = [tuple(np.concatenate([x, np.where(y >= 0, y + shift, -1)]) for x, y, shift in zip(a, b, (n, n, 0)))]
        l, r = np.array([1, 0, -1, -1]), np.array([2, 3, -1, -1])
        ranges.insert(50, (l, r, word(l)))
    off = np.concatenate([[0], np.cumsum([len(x[0]) for x in ranges])]).astype(np.int32)
    cat = lambda i, rel: np.concatenate([np.where(x[i] >= 0, x[i] + (o if rel else 0), -1) for x, o in zip(ranges, off)]).astype(np.int32)
    bad = synth.TreeBatch(off, cat(0, True), cat(1, True), cat(2, False))
    assert (bad.n_nodes + bad.n_trees) % 2 == 0 and (bad.left < 0).sum() * 2 == bad.n_nodes + bad.n_trees
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        binding.tl_set_keep_gates(net.ctx, True)
        binding.tl_set_async_backward(net.ctx, mode)
        for trees, expect in ((good, binding.TL_OK), (bad, binding.TL_ESTRUCT), (good, binding.TL_OK)):
            b = net.load(trees)
            net.forward()
            code = binding.TL_OK
            try:
                d_x = binding.tl_backward(net.ctx, b, torch.ones((trees.n_nodes, H), device="cuda"), params.embed_dim)["d_x"]
            except binding.TLError as e:
                code = e.code
            assert code == (expect if mode <= 0 else binding.TL_OK)
            assert binding.tl_status(net.ctx) == expect
            assert expect != binding.TL_OK or bool(torch.isfinite(d_x).all())
    finally:
        net.close()


def test_captured_backward_after_a_smaller_one():
    """A context that has evaluated more nodes than the tables hold: the first backward pass, of a small batch, allocates for all that they hold, so that a larger
    batch's can be recorded."""
    H, E = 512, 16
    params, huge = make("lstm", H, 1300, [4096] * 52, ["balanced"] * 52, E)
    assert huge.n_nodes * H * 20 >= 1 << 32
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        binding.tl_set_keep_gates(net.ctx, True)
        binding.tl_set_async_backward(net.ctx, 1)
        net.load(huge)
        net.forward()

        for n_trees, graphed in ((2, False), (60, True), (60, False)):
            print("case back captured after a smaller one", n_trees, graphed, flush=True)
            trees = synth.make_trees(1301, [20] * n_trees, ["random"] * n_trees, 50)
            b = net.load(trees)
            g = torch.ones((trees.n_nodes, H), device="cuda")
            net.forward()
            torch.cuda.synchronize()
            if graphed:
                graph, recorded = replayed(lambda: binding.tl_backward(net.ctx, b, g, E)["d_x"])
                graph.replay()
                torch.cuda.synchronize()
                recorded = recorded.clone()
            else:
                got = binding.tl_backward(net.ctx, b, g, E)["d_x"]
        assert binding.tl_status(net.ctx) == 0
        assert torch.equal(recorded, got)
    finally:
        net.close()


@pytest.mark.parametrize("cell", ["lstm", "rnn"])
def test_a_single_small_tree_is_not_slower_than_four(cell):
    """What a backward pass clears and packs does not depend on the number of nodes, so a batch of a few of them must not get a few workgroups for it."""
    H = 512
    us = []
    for counts in ([5], [5, 34, 17, 46]):
        params, trees = make(cell, H, 1310, counts, ["random"] * len(counts), 100)
        print("case back single small tree", cell, counts, flush=True)
        net = binding.TreeNet(params, scheduler="dataflow")
        try:
            b = net.load(trees)
            binding.tl_set_keep_gates(net.ctx, True)
            net.forward()
            g = torch.ones((trees.n_nodes, H), device="cuda")
            times = []
            for _ in range(30):
                begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                begin.record()
                binding.tl_backward(net.ctx, b, g, params.embed_dim)
                end.record()
                torch.cuda.synchronize()
                times.append(begin.elapsed_time(end) * 1e3)
            us.append(sorted(times)[10])
        finally:
            net.close()
    print(us, flush=True)
    assert us[0] < 1.1 * us[1], us
