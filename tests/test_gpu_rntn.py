"""The fp32 RNTN cell, whose operands are split into two fp16 terms, at the sizes where its tiles, slices, paddings and scales
can go wrong.

Tolerance: two terms hold a value to 2^-23 of itself (2^-38 of the largest of its row or column where it is far below that), a
product of two is off by 2^-21 at most; the sums of at most 2d (2d + 1) / 2 products here are of order one.  2e-5 relative + 2e-6
absolute is what the split TreeLSTM cells are tested with."""
import numpy as np
import pytest

import oracle
from paper_1809_00832_amd import binding, synth

pytestmark = pytest.mark.gpu
RTOL, ATOL = 2e-5, 2e-6


def run(params, trees, sched):
    net = binding.TreeNet(params, scheduler=sched)
    try:
        out = net.run(trees)
        for _ in range(2):
            net.batch["h"].fill_(float("nan"))
            net.forward()
            assert binding.tl_status(net.ctx) == 0
            assert np.array_equal(net.batch["h"].cpu().numpy(), out["h"], equal_nan=True)
        return out
    finally:
        net.close()


def check(got, ref):
    for key in ("h", "h_root"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)


@pytest.mark.parametrize("sched", ["dataflow", "level_device", "ready", "level_host"])
@pytest.mark.parametrize("d", [1, 7, 8, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 95, 96, 97, 128])
def test_sizes_at_the_edges_of_the_slices(d, sched):
    print("case rntn split sizes", d, sched, flush=True)
    params = synth.make_rnn_params(700 + d, synth.CELL_RNTN, 60, d, scale=0.7 / d ** 0.5)
    trees = synth.make_trees(701, [1, 2, 3, 1, 18, 40, 9, 33, 64], ["random", "chain", "balanced"] * 3, 60)
    check(run(params, trees, sched), oracle.forward_params(params, trees, n_threads=8))


@pytest.mark.parametrize("d", [1, 7, 8, 12, 16, 17, 20, 28, 31, 32, 33, 36, 48, 49, 60, 63, 64, 65, 80, 95, 96, 97, 128])
def test_every_scheduler_gives_the_same_bits(d):
    """Classes, k-steps of the linear term and parts are added in one order, in tiles of any size and by one wave a unit."""
    print("case rntn bits", d, flush=True)
    params = synth.make_rnn_params(705 + d, synth.CELL_RNTN, 60, d, scale=0.7 / d ** 0.5)
    trees = synth.make_trees(706, [1, 2, 40, 1, 18, 70, 9, 33, 64] * 6, ["random", "chain", "balanced"] * 18, 60)
    first = run(params, trees, "level_device")
    for sched in ("dataflow", "ready", "ready_priority", "level_host"):
        got = run(params, trees, sched)
        for key in ("h", "h_root"):
            assert np.array_equal(got[key], first[key]), (sched, key)


@pytest.mark.parametrize("sched", ["dataflow", "level_device"])
def test_rows_and_columns_of_very_different_size(sched):
    """Every embedding row and every column of a slice is scaled for itself: sizes four powers of ten apart side by side (the
    sums of absolute products reach 100, of which 2^-21 is left uncertain per product: hence the absolute tolerance)."""
    print("case rntn split scales", sched, flush=True)
    d = 40
    p = synth.make_rnn_params(710, synth.CELL_RNTN, 60, d, scale=0.1)
    rng = np.random.default_rng(1)
    p.v *= (10.0 ** rng.uniform(-3, 0, (d, 1, 1))).astype(np.float32)
    p.u *= (10.0 ** rng.uniform(-3, 0.5, d)).astype(np.float32)
    p.emb *= (10 * 10.0 ** rng.uniform(-4, 0.3, p.emb.shape[0])).astype(np.float32)[:, None]
    trees = synth.make_trees(711, [30, 8, 1, 21], ["random", "chain", "random", "balanced"], 60)
    got, ref = run(p, trees, sched), oracle.forward_params(p, trees, n_threads=8)
    assert np.abs(ref["h"][trees.left >= 0]).max() > 0.5
    np.testing.assert_allclose(got["h"], ref["h"], rtol=RTOL, atol=1e-5)


@pytest.mark.parametrize("sched", ["dataflow", "level_device", "ready"])
@pytest.mark.parametrize("where", ["v", "u", "emb"])
def test_infinities_are_summed_in_fp32(where, sched):
    """An infinity has no two terms; its sums are taken from the parameters as given."""
    print("case rntn infinity", where, sched, flush=True)
    d = 24
    p = synth.make_rnn_params(720, synth.CELL_RNTN, 30, d, scale=0.02)       # (sums of absolute products of order one)
    p.emb[:] = np.abs(p.emb) + 0.1                      # (no sum of infinities of both signs, which is a NaN)
    if where == "v":
        p.v[5, 3, 30] = np.inf
    elif where == "u":
        p.u[3, 5] = np.inf
    else:
        p.emb[::3, 5] = np.inf
        p.v[:] = np.abs(p.v)
        p.u[:] = np.abs(p.u)
    trees = synth.make_trees(721, [12, 5, 1, 20], ["random"] * 4, 30)
    with np.errstate(all="ignore"):
        ref = oracle.forward_params(p, trees, n_threads=8)
    got = run(p, trees, sched)
    ok = ~np.isnan(ref["h"])
    assert (np.abs(ref["h"][trees.left >= 0][:, 5]) == 1).any()
    np.testing.assert_allclose(got["h"][ok], ref["h"][ok], rtol=RTOL, atol=ATOL)


@pytest.mark.parametrize("cell,sched", [("rntn", "dataflow"), ("rntn", "level_device"), ("rntn", "level_host"), ("rnn", "dataflow")])
def test_sums_that_overflow_only_when_scaled(cell, sched):
    """3e34 - 1.9e34 - 1.9e34: the first term is beyond the largest number once it is scaled by 2^14, the others are not.  The sum
    is negative, so every internal node over two leaves is -1 there."""
    print("case scaled overflow", cell, sched, flush=True)
    d = 64 if cell == "rnn" else 16
    p = synth.make_rnn_params(735, synth.CELL_RNTN if cell == "rntn" else synth.CELL_TREERNN, 2, d, scale=0.01)
    if cell == "rntn":
        p.emb[:] = 1
        p.v[3, 0, 0], p.v[3, 1, 1], p.v[3, 2, 2] = 3e34, -1.9e34, -1.9e34
    else:                                               # three different quarters of the K axis
        p.emb[:, 0] = 6e34, 3.9e34
        p.emb[1, 40] = 3.9e34
        p.u[:] = 0
        p.u[0, 3], p.u[d, 3], p.u[d + 40, 3] = 1, -1, -1
    trees = synth.make_trees(736, [2] * 20, ["random"] * 20, 2)
    trees.word[trees.left[trees.left >= 0]], trees.word[trees.right[trees.left >= 0]] = 0, 1
    ref = oracle.forward_params(p, trees, n_threads=4)
    got = run(p, trees, sched)
    inner = trees.left >= 0
    assert (ref["h"][inner, 3] == -1).all()
    assert (got["h"][inner, 3] == -1).all()
    np.testing.assert_allclose(got["h"][~inner], ref["h"][~inner])


@pytest.mark.parametrize("where", ["emb", "v", "u", "b"])
@pytest.mark.parametrize("cell,d", [("rntn", 24), ("rntn", 33), ("rnn", 40)])
def test_a_nan_of_32_ones_ends_no_forward(cell, d, where):
    """The data-flow scheduler reads all ones as "not written yet".  A NaN that happens to have these bits gives what it gives
    level by level (leaves hold it as it is; the clamp in tanh makes a number of the sums over it), and nodes not above it
    are those of the checker."""
    if cell == "rnn" and where == "v":
        pytest.skip("TreeRNN has no tensor")
    print("case nan of ones", cell, d, where, flush=True)
    p = synth.make_rnn_params(730, synth.CELL_RNTN if cell == "rntn" else synth.CELL_TREERNN, 30, d, scale=0.1)
    a = getattr(p, where)
    a.view(np.uint32)[{"emb": (slice(4, 8), slice(0, 3)), "v": (5, 3, 30 % d), "u": (3, 5), "b": 5}[where]] = 0xFFFFFFFF
    trees = synth.make_trees(731, [12, 5, 1, 20, 40], ["random", "chain", "random", "balanced", "chain"], 30)
    with np.errstate(all="ignore"):
        ref = oracle.forward_params(p, trees, n_threads=8)
    got = {}
    for sched in ("level_device", "dataflow"):
        net = binding.TreeNet(p, scheduler=sched, spin_limit=20000)
        try:
            got[sched] = net.run(trees)
        finally:
            net.close()
        ok = ~np.isnan(ref["h"])
        if where != "emb":                              # (one unit of every node is affected, and what stands on it)
            ok[:] = False
            ok[trees.left < 0] = True
        assert ok.any() and np.isnan(ref["h"]).any()
        np.testing.assert_allclose(got[sched]["h"][ok], ref["h"][ok], rtol=RTOL, atol=4e-6)
    for key in ("h", "h_root"):
        np.testing.assert_allclose(got["dataflow"][key], got["level_device"][key], rtol=RTOL, atol=4e-6, equal_nan=True, err_msg=key)


# ---- TreeRNN under the data-flow scheduler: the split cell with rows of any scale ------------------------------------
@pytest.mark.parametrize("n_trees", [9, 700])           # one column group per workgroup, and two
@pytest.mark.parametrize("H", [1, 15, 16, 17, 33, 64, 65, 129, 256, 301, 479, 512])
def test_treernn_sizes_at_the_edges_of_the_tiles(H, n_trees):
    print("case rnn split sizes", H, n_trees, flush=True)
    params = synth.make_rnn_params(740 + H, synth.CELL_TREERNN, 60, H, scale=1.0 / H ** 0.5)
    params.emb *= np.float32(H ** 0.5)
    trees = synth.make_trees(741, ([1, 2, 3, 1, 18, 40, 9, 33, 64] * 78)[:n_trees], (["random", "chain", "balanced"] * 234)[:n_trees], 60)
    got, ref = run(params, trees, "dataflow"), oracle.forward_params(params, trees, n_threads=8)
    # (sums of up to 1 024 products of which those of leaves reach 1)
    for key in ("h", "h_root"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=4e-6, err_msg=key)


def test_treernn_rows_and_columns_of_very_different_size():
    """Leaves keep the scale of their embedding row: sizes from 1e-3 to 1e3 side by side, columns of the weights from 1e-6 to 1."""
    print("case rnn split scales", flush=True)
    H = 72
    p = synth.make_rnn_params(750, synth.CELL_TREERNN, 60, H, scale=0.1)
    rng = np.random.default_rng(2)
    p.u *= (10.0 ** rng.uniform(-6, 0, H)).astype(np.float32)
    p.emb *= (10.0 ** rng.uniform(-3, 1, p.emb.shape[0])).astype(np.float32)[:, None]
    p.emb[::9] *= 1e3
    trees = synth.make_trees(751, [30, 8, 1, 21], ["random", "chain", "random", "balanced"], 60)
    got, ref = run(p, trees, "dataflow"), oracle.forward_params(p, trees, n_threads=8)
    # a sum over a row of 1e3 carries 2^-21 of its absolute products (144 of up to 100): 7e-3 where it does not saturate
    big = np.abs(ref["h"]).max(axis=1) > 20
    inner = trees.left >= 0
    over_big = np.zeros(trees.n_nodes, dtype=bool)
    over_big[inner] = big[trees.left[inner]] | big[trees.right[inner]]
    tainted = over_big.copy()                           # and what stands on such a node
    for _ in range(40):
        tainted[inner] |= tainted[trees.left[inner]] | tainted[trees.right[inner]]
    assert tainted.any() and not tainted[inner].all()
    np.testing.assert_allclose(got["h"][~tainted], ref["h"][~tainted], rtol=RTOL, atol=4e-6)
    np.testing.assert_allclose(got["h"][tainted], ref["h"][tainted], rtol=RTOL, atol=7e-3)


@pytest.mark.parametrize("where", ["u", "emb"])
def test_treernn_infinities_are_summed_in_fp32(where):
    print("case rnn infinity", where, flush=True)
    H = 40
    p = synth.make_rnn_params(760, synth.CELL_TREERNN, 30, H, scale=0.1)
    p.emb[:] = np.abs(p.emb) + 0.1
    p.u[:] = np.abs(p.u)
    if where == "u":
        p.u[3, 5] = np.inf
    else:
        p.emb[::3, 5] = np.inf
    trees = synth.make_trees(761, [12, 5, 1, 20], ["random"] * 4, 30)
    with np.errstate(all="ignore"):
        ref = oracle.forward_params(p, trees, n_threads=8)
    got = run(p, trees, "dataflow")
    assert not np.isnan(ref["h"]).any() and (ref["h"][trees.left >= 0][:, 5] == 1).any()
    np.testing.assert_allclose(got["h"], ref["h"], rtol=RTOL, atol=4e-6)


# ---- both cells: sets of workgroups, their places, and the choice of the kernel ---------------------------------------
def small_params(cell, d, seed):
    p = synth.make_rnn_params(seed, synth.CELL_RNTN if cell == "rntn" else synth.CELL_TREERNN, 60, d, scale=(0.7 if cell == "rntn" else 1.0) / d ** 0.5)
    return p


@pytest.mark.parametrize("cell,d,n_trees,leaves", [("rnn", 80, 51, 9), ("rnn", 80, 52, 9), ("rnn", 96, 42, 9), ("rnn", 96, 43, 9), ("rnn", 96, 86, 9), ("rnn", 208, 19, 20),
                                                   ("rnn", 208, 20, 20), ("rnn", 224, 18, 20), ("rnn", 100, 380, 40), ("rnn", 100, 400, 40), ("rnn", 40, 380, 40), ("rnn", 40, 400, 40),
                                                   ("rntn", 20, 51, 9), ("rntn", 20, 52, 9), ("rntn", 20, 51, 190), ("rntn", 20, 52, 190), ("rntn", 32, 33, 9), ("rntn", 36, 29, 9),
                                                   ("rntn", 12, 90, 90), ("rntn", 12, 110, 90)])
def test_sets_of_workgroups_on_both_sides_of_the_lines(cell, d, n_trees, leaves):
    """One workgroup a CU or two, one column group per workgroup or two, sets inside one domain or on all of them: as many trees as
    there are sets and one more, batches on both sides of the line in nodes.  Every node is evaluated once, by all of its columns."""
    print("case sets", cell, d, n_trees, leaves, flush=True)
    p = small_params(cell, d, 900 + d)
    trees = synth.make_trees(901, [leaves - t % 5 for t in range(n_trees)], (["random", "chain", "balanced"] * n_trees)[:n_trees], 60)
    got, ref = run(p, trees, "dataflow"), oracle.forward_params(p, trees, n_threads=8)
    for key in ("h", "h_root"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=4e-6, err_msg=key)


@pytest.mark.parametrize("cell,d,line", [("rnn", 33, 1024), ("rnn", 100, 1024), ("rntn", 24, 2048), ("rntn", 72, 1536)])
def test_few_large_trees_of_either_kind_one_after_the_other(cell, d, line):
    """Few trees of more nodes than the line: both kernels are launched and the device picks.  Bushy trees, then deep ones, then bushy
    ones again through one context (rows marked for a kernel that did not run become leaves and the other way round), and
    trees just below the line, against the checker.  TreeRNN, whose two kernels sum in different orders: bushy trees have the
    level scheduler's bits, deep ones and those below the line have not."""
    print("case few large trees", cell, d, flush=True)
    p = small_params(cell, d, 910 + d)
    L = line // 2 + 1                                   # 2 L - 1 nodes, one more than the line
    nets = {s: binding.TreeNet(p, scheduler=s) for s in ("dataflow", "level_device")}
    try:
        for i, (shape, leaves) in enumerate([("balanced", L + 9), ("chain", L), ("random", L + 60), ("balanced", L - 1), ("balanced", L)]):
            trees = synth.make_trees(911 + i, [leaves] * 3, [shape] * 3, 60)
            ref = oracle.forward_params(p, trees, n_threads=8)
            got = {s: n.run(trees) for s, n in nets.items()}
            for s in got:
                for key in ("h", "h_root"):
                    np.testing.assert_allclose(got[s][key], ref[key], rtol=RTOL, atol=4e-6, err_msg="%s %s %s" % (s, shape, key))
            if cell == "rnn":
                assert np.array_equal(got["dataflow"]["h"], got["level_device"]["h"]) == (shape != "chain" and leaves >= L), (shape, leaves)
    finally:
        for n in nets.values():
            n.close()


# ---- RNTN: the backward pass in one kernel (d <= 96) -------------------------------------------------------------------
def rntn_gradients(params, trees, g_h, modes=(0, 1)):
    import torch
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        b = net.load(trees)
        net.forward()
        out = {}
        for mode in modes:
            binding.tl_set_async_backward(net.ctx, mode)
            got = binding.tl_backward(net.ctx, b, torch.from_numpy(g_h).cuda(), params.embed_dim, rntn=True)
            torch.cuda.synchronize()
            assert binding.tl_status(net.ctx) == 0
            out[mode] = {k: v.cpu().numpy() for k, v in got.items()}
        h = b["h"].cpu().numpy()
    finally:
        net.close()
    with np.errstate(all="ignore"):
        ref = oracle.backward(params, trees, h, None, g_h)
    ref["d_w_leaf"] = ref.pop("d_v")
    return out, ref


@pytest.mark.parametrize("d,n_trees", [(d, 9) for d in (1, 7, 8, 16, 17, 31, 32, 33, 48, 49, 64, 65, 80, 95, 96, 97)] + [(16, 150), (33, 150), (64, 40)])
def test_rntn_gradients_at_the_edges_of_the_blocks(d, n_trees):
    """Against the checker: products to 2^-21, sums of at most 2d d of them of order one, carried down up to 33 heights (1e-4 of the
    largest, the figure that the other gradients are tested with)."""
    print("case rntn backward sizes", d, n_trees, flush=True)
    params = synth.make_rnn_params(770 + d, synth.CELL_RNTN, 60, d, scale=0.3 / d ** 0.5)
    trees = synth.make_trees(771, ([1, 2, 3, 1, 18, 30, 9, 33, 16] * 17)[:n_trees], (["random", "chain", "balanced"] * 51)[:n_trees], 60)
    g_h = np.random.default_rng(d).standard_normal((trees.n_nodes, d)).astype(np.float32)
    out, ref = rntn_gradients(params, trees, g_h)
    assert np.array_equal(out[0]["d_x"], out[1]["d_x"])
    for k in ref:
        np.testing.assert_allclose(out[0][k], ref[k].reshape(out[0][k].shape), rtol=1e-4, atol=1e-4 * max(1e-3, float(np.abs(ref[k]).max())), err_msg=k)


@pytest.mark.parametrize("d", [20, 48, 96])
def test_rntn_backward_in_every_mode(d):
    """tl_set_async_backward and RNTN: -1 takes launches per height (fp32 instructions, another order of summation: the same
    gradients to rounding, other bits), 0 and 1 the one kernel, and a malformed batch is reported by the call in every mode.
    Modes alternate on one context, with an update in between: each finds its packed matrix and its workspace."""
    import torch
    print("case rntn backward modes", d, flush=True)
    params = synth.make_rnn_params(790 + d, synth.CELL_RNTN, 60, d, scale=0.3 / d ** 0.5)
    trees = synth.make_trees(791, [1, 2, 30, 1, 18, 33, 9], ["random", "chain", "balanced", "random", "chain", "random", "balanced"], 60)
    g_h = np.random.default_rng(d).standard_normal((trees.n_nodes, d)).astype(np.float32)
    dev_g = torch.from_numpy(g_h).cuda()
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        b = net.load(trees)
        bad = dict(b)
        bad["left"] = b["left"].clone()
        bad["left"][trees.n_nodes - 1] = 0              # the last leaf gets one child, and that in another tree
        for step in range(2):
            net.forward()
            out = {}
            for mode in (0, -1, 1):
                binding.tl_set_async_backward(net.ctx, mode)
                out[mode] = {k: v.cpu().numpy() for k, v in binding.tl_backward(net.ctx, b, dev_g, d, rntn=True).items()}
                assert binding.tl_status(net.ctx) == 0
                with pytest.raises(binding.TLError) as e:
                    binding.tl_backward(net.ctx, bad, dev_g, d, rntn=True)
                assert e.value.code == binding.TL_ESTRUCT and binding.tl_status(net.ctx) == binding.TL_ESTRUCT
            p = binding.tl_get_params(net.ctx, 60, d, d, cell=params.cell)
            ref = oracle.backward(synth.Params(params.cell, 60, d, d, p["emb"].cpu().numpy(), None, None, p["u"].cpu().numpy(), p["b"].cpu().numpy(),
                                               p["w_leaf"].cpu().numpy()), trees, b["h"].cpu().numpy(), None, g_h)
            ref["d_w_leaf"] = ref.pop("d_v")
            assert np.array_equal(out[0]["d_x"], out[1]["d_x"])
            assert not np.array_equal(out[-1]["d_x"], out[0]["d_x"]), "launches per height were expected to run"
            for mode in out:
                for k in ref:
                    np.testing.assert_allclose(out[mode][k], ref[k].reshape(out[mode][k].shape), rtol=1e-4, atol=1e-4 * max(1e-3, float(np.abs(ref[k]).max())),
                                               err_msg="step %d mode %d %s" % (step, mode, k))
            binding.tl_sgd_update(net.ctx, 1e-2, b, {k: torch.from_numpy(v).cuda() for k, v in out[0].items()})
    finally:
        net.close()


@pytest.mark.parametrize("what", ["scales", "infinite weight", "nan gradient"])
def test_rntn_gradients_outside_the_ordinary_range(what):
    """Gradients are factors as they are, of any magnitude; an infinite operand is met in fp32; a NaN stays where it belongs."""
    print("case rntn backward range", what, flush=True)
    d = 24
    params = synth.make_rnn_params(780, synth.CELL_RNTN, 40, d, scale=0.05)
    params.emb[:] = np.abs(params.emb) + 0.1
    trees = synth.make_trees(781, [12, 5, 1, 20], ["random", "chain", "random", "balanced"], 40)
    rng = np.random.default_rng(3)
    g_h = rng.standard_normal((trees.n_nodes, d)).astype(np.float32)
    tree = np.searchsorted(trees.tree_off, np.arange(trees.n_nodes), side="right") - 1
    if what == "scales":
        g_h *= np.array([1e-25, 1e12, 1.0, 1e-8], dtype=np.float32)[tree][:, None]       # (a tree's gradients do not meet another's in d_x)
    elif what == "infinite weight":
        params.v[5, 3, 30] = np.inf
    else:
        g_h[trees.tree_off[1], 7] = np.nan
    out, ref = rntn_gradients(params, trees, g_h)
    got, want = out[0]["d_x"], ref["d_x"]
    assert np.array_equal(np.isnan(got), np.isnan(want))
    for t in range(4):
        m = (tree == t)[:, None] & np.isfinite(want)
        if m.any():
            np.testing.assert_allclose(got[m], want[m], rtol=1e-4, atol=1e-4 * float(np.abs(want[m]).max()), err_msg="tree %d" % t)


def test_rntn_gradients_of_weights_near_the_largest_number():
    """Weights of up to 2e34 beside states of 5e-18: a product of scaled terms and the column's scale alone would be infinite, the
    gradient of an operand (sums of 2d d such products, up to 1e17) is not."""
    print("case rntn backward, largest weights", flush=True)
    d = 16
    params = synth.make_rnn_params(795, synth.CELL_RNTN, 40, d, scale=0.05)
    params.v *= np.float32(4e35)
    params.emb *= np.float32(1e-16)
    trees = synth.make_trees(796, [2] * 40, ["random"] * 40, 40)
    g_h = np.random.default_rng(4).standard_normal((trees.n_nodes, d)).astype(np.float32)
    out, ref = rntn_gradients(params, trees, g_h)
    want = ref["d_x"]
    assert np.isfinite(want).all() and np.abs(want).max() > 1e16
    np.testing.assert_allclose(out[0]["d_x"], want, rtol=1e-4, atol=1e-4 * float(np.abs(want).max()))


# ---- both cells: after an update --------------------------------------------------------------------------------------
@pytest.mark.parametrize("cell,d", [("rntn", 20), ("rntn", 64), ("rntn", 72), ("rntn", 100), ("rnn", 24), ("rnn", 150), ("rnn", 272)])
def test_after_an_update_a_context_is_like_a_fresh_one(cell, d):
    """tl_sgd_update rebuilds every packed form of the parameters: forward and operand gradient have the bits of a context made from the
    updated parameters, with steps that change the largest magnitudes of columns by powers of ten."""
    import torch
    print("case update", cell, d, flush=True)
    p = small_params(cell, d, 920 + d)
    trees = synth.make_trees(921, [30, 8, 1, 21, 2, 60], ["random", "chain", "random", "balanced", "random", "chain"], 60)
    gen = torch.Generator(device="cuda").manual_seed(6)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    g_h = rand(trees.n_nodes, d)

    def both(net):
        net.forward()
        g = binding.tl_backward(net.ctx, net.batch, g_h, d, rntn=cell == "rntn")
        assert binding.tl_status(net.ctx) == 0
        return {"h": net.batch["h"].cpu().numpy(), "h_root": net.batch["h_root"].cpu().numpy(), **{k: v.cpu().numpy() for k, v in g.items()}}

    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        net.load(trees)
        before = both(net)
        grads = dict(d_u=rand(2 * d, d) * torch.logspace(-5, 0, d, device="cuda"), d_b=rand(d), d_x=rand(trees.n_nodes, d))
        if cell == "rntn":
            grads["d_w_leaf"] = rand(d, 2 * d, 2 * d) * torch.logspace(0, -5, d, device="cuda")[:, None, None]
        binding.tl_sgd_update(net.ctx, 0.05, net.batch, grads)
        new = {k: v.cpu().numpy() for k, v in binding.tl_get_params(net.ctx, 60, d, d, cell=p.cell).items()}
        after = both(net)
    finally:
        net.close()
    assert np.abs(after["h"] - before["h"]).max() > 1e-2
    q = synth.Params(p.cell, 60, d, d, new["emb"], None, None, new["u"], new["b"], new.get("w_leaf"))
    fresh = binding.TreeNet(q, scheduler="dataflow")
    try:
        fresh.load(trees)
        want = both(fresh)
    finally:
        fresh.close()
    for key in ("h", "h_root", "d_x"):
        assert np.array_equal(after[key], want[key]), key
    for key in ("d_u", "d_b") + (("d_w_leaf",) if cell == "rntn" else ()):      # (sums over the nodes by atomics)
        np.testing.assert_allclose(after[key], want[key], rtol=1e-4, atol=2e-5 * float(np.abs(want[key]).max()), err_msg=key)
