"""Error paths of the C ABI on the GPU.  Every case is rejected by the host or by the structure pass before any
cell reads through a bad index, or ends in the scheduler's bounded wait: all kernels exit normally."""
import numpy as np
import pytest
import torch

from paper_1809_00832_amd import binding, synth
from paper_1809_00832_amd.synth import TreeBatch

pytestmark = pytest.mark.gpu
SCHEDULERS = ["level_host", "level_device", "ready", "ready_priority", "dataflow"]


def run_expect(params, trees, sched, expect, **kw):
    net = binding.TreeNet(params, scheduler=sched, **kw)
    try:
        net.load(trees)
        net.batch["h"].zero_()
        try:
            net.forward()
            code = binding.tl_status(net.ctx)
        except binding.TLError as e:         # rejected by the host before anything was enqueued
            code = e.code
        assert code == expect, "%s: got %s, expected %s" % (sched, binding.tl_strerror(code), binding.tl_strerror(expect))
        # the context stays usable: a good batch afterwards evaluates without error
        good = synth.make_trees(3, [4, 2], ["random"] * 2, params.vocab)
        net.load(good)
        net.forward()
        assert binding.tl_status(net.ctx) == binding.TL_OK
        assert torch.isfinite(net.batch["h"]).all()
    finally:
        net.close()


def small_params():
    return synth.make_treelstm_params(1, 50, 8, 32, "xavier")


def good_trees():
    return synth.make_trees(2, [5, 3, 6], ["random"] * 3, 50)


@pytest.mark.parametrize("sched", SCHEDULERS)
def test_structure_errors_are_latched(sched):
    print("case structure errors", sched, flush=True)
    p = small_params()
    t = good_trees()
    off = [int(x) for x in t.tree_off]

    def variant(**chg):
        d = dict(tree_off=t.tree_off.copy(), left=t.left.copy(), right=t.right.copy(), word=t.word.copy())
        for k, f in chg.items():
            f(d[k])
        return TreeBatch(**d)

    internal = int(np.flatnonzero(t.left >= 0)[0])
    leaf = int(np.flatnonzero(t.left < 0)[0])
    cases = {
        "child in another tree": variant(left=lambda a: a.__setitem__(off[0], off[1])),
        "child index beyond the batch": variant(right=lambda a: a.__setitem__(internal, t.n_nodes + 5)),
        "one child missing": variant(right=lambda a: a.__setitem__(internal, -1)),
        "node with two parents": variant(left=lambda a: a.__setitem__(internal, int(t.right[internal]))),
        "word id beyond the vocabulary": variant(word=lambda a: a.__setitem__(leaf, 50)),
        "negative word id": variant(word=lambda a: a.__setitem__(leaf, -1)),
        "offsets not ascending": variant(tree_off=lambda a: a.__setitem__(1, off[2])),
        "last offset is not the node count": variant(tree_off=lambda a: a.__setitem__(3, off[3] - 1)),
    }
    for what, bad in cases.items():
        print("   ", what, flush=True)
        run_expect(p, bad, sched, binding.TL_ESTRUCT)


def cyclic_batch():
    """One tree range holding a proper 3-node tree plus a detached 2-cycle with two leaves:
    0 = (1, 2), 3 = (4, 5), 4 = (3, 6); leaves 1, 2, 5, 6.  One root, every node one parent, counts consistent."""
    left = np.array([1, -1, -1, 4, 3, -1, -1], np.int32)
    right = np.array([2, -1, -1, 5, 6, -1, -1], np.int32)
    word = np.array([-1, 3, 4, -1, -1, 5, 6], np.int32)
    return TreeBatch(np.array([0, 7], np.int32), left, right, word)


@pytest.mark.parametrize("sched", SCHEDULERS)
def test_unreachable_nodes(sched):
    """Level schedulers (and validate=1) see that the bottom-up sweep does not reach every node; the ready
    scheduler without validation runs out of its (here: tiny) spin budget and reports a stall."""
    print("case cycle", sched, flush=True)
    p = small_params()
    if sched.startswith("ready"):
        run_expect(p, cyclic_batch(), sched, binding.TL_ESTALL, spin_limit=2000)
        run_expect(p, cyclic_batch(), sched, binding.TL_ESTRUCT, validate=1)
    else:
        run_expect(p, cyclic_batch(), sched, binding.TL_ESTRUCT)


def test_host_side_argument_checks():
    p = small_params()
    t = good_trees()
    net = binding.TreeNet(p, scheduler="ready")
    try:
        b = net.load(t)
        L = binding.lib()
        args = [b["tree_off"], b["left"], b["right"], b["word"], b["h"], b["c"], b["h_root"], b["c_root"], b["root"]]
        ptr = [x.data_ptr() for x in args]
        st = torch.cuda.current_stream().cuda_stream
        assert L.tl_forward(net.ctx, 0, b["N"], *ptr, st) == binding.TL_EINVAL
        assert L.tl_forward(net.ctx, 0, 0, *([None] * 9), st) == binding.TL_OK                      # an empty batch is a no-op
        assert binding.tl_status(net.ctx) == binding.TL_OK
        assert binding.tl_last_stats(net.ctx)["n_workgroups"] == 0
        assert L.tl_forward(net.ctx, b["B"], b["B"] - 1, *ptr, st) == binding.TL_EINVAL
        assert L.tl_forward(net.ctx, b["B"], b["N"], None, *ptr[1:], st) == binding.TL_EINVAL
        assert L.tl_forward(net.ctx, b["B"], b["N"], *ptr[:5], None, *ptr[6:], st) == binding.TL_EINVAL   # c missing
        assert L.tl_forward(net.ctx, b["B"], b["N"] - 1, *ptr, st) == binding.TL_ESTRUCT             # N + B odd
        assert L.tl_forward(None, b["B"], b["N"], *ptr, st) == binding.TL_EINVAL
        assert L.tl_forward(net.ctx, b["B"], b["N"], *ptr, st) == binding.TL_OK
        assert binding.tl_status(net.ctx) == binding.TL_OK
    finally:
        net.close()
    with pytest.raises(binding.TLError):
        binding.tl_create(7, 0, 0, 10, 4, 4, torch.zeros(10, 4, device="cuda"))
    with pytest.raises(binding.TLError):          # TreeRNN needs embed_dim == hidden
        z = torch.zeros(8, 8, device="cuda")
        binding.tl_create(binding.TL_TREERNN, 0, 0, 8, 8, 4, z, u=z, b=z)


@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("name", ["sentence", "throughput", "treernn"])
def test_results_do_not_depend_on_the_schedule(name, precision):
    """Every data path sums a node's contraction in the same order (four quarters of the K axis,
    each in k order, added in quarter order), whatever rows share its tile.  So the schedulers agree bit
    for bit with each other and from run to run, although the ready scheduler forms different tiles every time.
    (Same recursion, different execution order, identical numbers: the claim of Section 5's numerical check.)
    One exception: in fp32 the data-flow scheduler sums the internal nodes of a TreeLSTM or a TreeRNN from operands split into two
    fp16 terms; it still repeats its own bits from run to run, and agrees with the others to rounding."""
    print("case determinism", name, precision, flush=True)
    w = synth.workload(name)
    outs = []
    for sched in ("ready", "level_device", "level_host", "ready_priority", "dataflow"):
        net = binding.TreeNet(w.params, scheduler=sched, precision=binding.TL_F32 if precision == "f32" else binding.TL_BF16_IN)
        try:
            got = net.run(w.trees)
            outs.append((sched, got["h"].copy(), None if got["c"] is None else got["c"].copy()))
            for again in range(3):
                net.batch["h"].fill_(float("nan"))
                net.forward()
                assert binding.tl_status(net.ctx) == 0
                h2 = net.batch["h"].cpu().numpy()
                diff = int((h2 != got["h"]).sum())
                assert diff == 0, "%s run %d: %d elements differ from the first run, max %.3e" % (
                    sched, again, diff, np.abs(h2 - got["h"]).max())
        finally:
            net.close()
    for sched, h, c in outs[1:]:
        if sched == "dataflow" and precision == "f32":
            np.testing.assert_allclose(h, outs[0][1], rtol=2e-5, atol=2e-6, err_msg="dataflow vs ready: h")
            if c is not None:
                np.testing.assert_allclose(c, outs[0][2], rtol=2e-5, atol=2e-6, err_msg="dataflow vs ready: c")
            continue
        diff = int((h != outs[0][1]).sum())
        assert diff == 0, "%s vs ready: %d h elements differ, max %.3e" % (sched, diff, np.abs(h - outs[0][1]).max())
        assert c is None or np.array_equal(c, outs[0][2]), "%s vs ready: c differs" % sched


@pytest.mark.parametrize("sched", ["ready", "level_device", "ready_priority", "dataflow"])
def test_forward_replayed_from_a_hip_graph(sched):
    """tl_forward of the two device-scheduled variants makes no host round trip and clears its state with fill
    kernels, so it can be captured in a HIP graph.  Every replay, with eager work and synchronisation between
    replays and with new child states poisoned each time, must reproduce the eager result bit for bit."""
    print("case graph", sched, flush=True)
    w = synth.workload("sentence")
    net = binding.TreeNet(w.params, scheduler=sched)
    try:
        net.load(w.trees)
        net.forward()                                   # eager: also sizes the workspace, nothing is allocated later
        torch.cuda.synchronize()
        assert binding.tl_status(net.ctx) == 0
        eager_h = net.batch["h"].clone()
        eager_c = net.batch["c"].clone()
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.graph(graph, stream=side):
            net.forward()
        for it in range(4):
            net.batch["h"].fill_(float("nan"))
            net.batch["c"].fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(net.batch["h"], eager_h) and torch.equal(net.batch["c"], eager_c), "replay %d differs" % it
            scratch = torch.randn(1 << 16, device="cuda").sum().item()      # unrelated eager work between replays
            assert scratch == scratch
        assert binding.tl_status(net.ctx) == 0
    finally:
        net.close()


@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("sched", ["ready", "level_device", "ready_priority", "dataflow"])
@pytest.mark.parametrize("name,iters", [("throughput", 300), ("sentence", 300), ("stress", 20), ("mixed_small", 200)])
def test_many_forwards_give_the_same_bits(name, iters, sched, precision):
    """Many forwards of one batch through one context: every one ends without error and with exactly the bits of
    the first (tile composition, arrival order at the barriers and queue order differ from run to run).  The state
    arrays are poisoned before every checked forward, so a row that is read before it is written shows."""
    print("case soak", name, sched, precision, flush=True)
    w = synth.workload(name)
    net = binding.TreeNet(w.params, scheduler=sched, precision=binding.TL_F32 if precision == "f32" else binding.TL_BF16_IN)
    try:
        net.load(w.trees)
        net.forward()
        torch.cuda.synchronize()
        assert binding.tl_status(net.ctx) == 0
        h0, c0 = net.batch["h"].clone(), net.batch["c"].clone()
        bad = 0
        checked = 0
        for it in range(iters):
            check = it % 10 == 9 or iters <= 20
            if check:
                net.batch["h"].fill_(float("nan"))
                net.batch["c"].fill_(float("nan"))
            net.forward()
            if check:
                checked += 1
                bad += int(not (torch.equal(net.batch["h"], h0) and torch.equal(net.batch["c"], c0)))
        torch.cuda.synchronize()
        assert binding.tl_status(net.ctx) == 0
        assert bad == 0, "%d of %d checked forwards differ from the first" % (bad, checked)
    finally:
        net.close()


def batch_with_wrong_roots(n_good, leaves, vocab):
    """Good trees around two ranges whose counts add up while neither is a tree: 6 nodes with two roots, and 4 nodes that
    form a cycle and have none (every node has one parent at most, leaves and internal nodes are as many as they should be).
    What is wrong is found by whoever looks for the roots: under the data-flow scheduler workgroups of one slot, beside the others."""
    good = synth.make_trees(7, [leaves] * n_good, ["random", "balanced"] * (n_good // 2), vocab)
    two = (np.array([1, -1, -1, 4, -1, -1]), np.array([2, -1, -1, 5, -1, -1]))
    ring = (np.array([1, 0, -1, -1]), np.array([2, 3, -1, -1]))
    off, left, right, word = [0], [], [], []

    def add(l, r, w):
        base = off[-1]
        left.append(np.where(l >= 0, l + base, -1))
        right.append(np.where(r >= 0, r + base, -1))
        word.append(w)
        off.append(base + len(l))

    for t in range(n_good):
        if t == n_good // 3: add(*two, np.where(two[0] < 0, 3, -1))
        if t == 2 * n_good // 3: add(*ring, np.where(ring[0] < 0, 4, -1))
        lo, hi = int(good.tree_off[t]), int(good.tree_off[t + 1])
        rel = lambda a: np.where(a[lo:hi] >= 0, a[lo:hi] - lo, -1)
        add(rel(good.left), rel(good.right), good.word[lo:hi])
    cat = lambda a: np.concatenate(a).astype(np.int32)
    return TreeBatch(np.array(off, np.int32), cat(left), cat(right), cat(word))


@pytest.mark.parametrize("what", ["lstm", "lstm, large slots", "lstm bf16", "rnn", "rnn bf16"])
def test_errors_found_by_one_slot_beside_the_others(what):
    """A workgroup leaves as a whole: an error that another slot latches while a workgroup starts must not part its waves
    (their shares of the tables in LDS would be missing).  The batch is rejected, again and again, and the context goes on."""
    print("case errors beside other slots", what, flush=True)
    large = "large" in what
    H = 500 if large else 16
    p = synth.make_rnn_params(5, synth.CELL_TREERNN, 50, H, scale=0.4) if "rnn" in what else synth.make_treelstm_params(5, 50, 8, H, "xavier")
    bad = batch_with_wrong_roots(40 if large else 300, 1200 if large else 20, 50)
    assert (bad.n_nodes + bad.n_trees) % 2 == 0 and (bad.left < 0).sum() * 2 == bad.n_nodes + bad.n_trees
    kw = dict(precision=binding.TL_BF16_IN) if "bf16" in what else {}
    for _ in range(2 if large else 6):
        run_expect(p, bad, "dataflow", binding.TL_ESTRUCT, **kw)


@pytest.mark.parametrize("cell,H,mode", [("rntn", 16, 0), ("rntn", 16, 1), ("rnn", 520, 1), ("lstm", 520, 1)])
def test_backward_without_a_leaf_list(cell, H, mode):
    """No leaf has a valid word, so the leaf list holds nothing: where the call does not wait for the structure pass, no kernel behind it may look there."""
    print("case backward without a leaf list", cell, H, mode, flush=True)
    if cell == "lstm":
        p = synth.make_treelstm_params(1, 50, 8, H, "xavier")
    else:
        p = synth.make_rnn_params(5, synth.CELL_RNTN if cell == "rntn" else synth.CELL_TREERNN, 50, H, scale=0.02)
    t = good_trees()
    bad = TreeBatch(t.tree_off, t.left, t.right, np.full_like(t.word, 50))
    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        b = net.load(bad)
        binding.tl_set_keep_gates(net.ctx, True)
        binding.tl_set_async_backward(net.ctx, mode)
        net.forward()
        g_h = torch.ones((b["N"], H), device="cuda")
        code = binding.TL_OK
        try:
            binding.tl_backward(net.ctx, b, g_h, p.embed_dim, rntn=cell == "rntn")
        except binding.TLError as e:
            code = e.code
        assert code == (binding.TL_ESTRUCT if cell == "rntn" else binding.TL_OK)
        assert binding.tl_status(net.ctx) == binding.TL_ESTRUCT
    finally:
        net.close()


def batch_with_too_many_leaves(n_good):
    """Good trees around a range of three leaves without a parent: N + B stays even, and nothing but the number of leaves is wrong."""
    if n_good == 0:
        return TreeBatch(np.array([0, 3], np.int32), np.full(3, -1, np.int32), np.full(3, -1, np.int32), np.full(3, 7, np.int32))
    t = synth.make_trees(11, [6] * n_good, ["random"] * n_good, 50)
    cut = int(t.tree_off[n_good // 2])
    move = lambda a: np.where(a >= cut, a + 3, a)
    put = lambda a, v: np.concatenate([a[:cut], np.full(3, v), a[cut:]]).astype(np.int32)
    off = np.concatenate([t.tree_off[:n_good // 2 + 1], t.tree_off[n_good // 2:] + 3]).astype(np.int32)
    return TreeBatch(off, put(move(t.left), -1), put(move(t.right), -1), put(t.word, 7))


@pytest.mark.parametrize("n_good", [0, 40])
@pytest.mark.parametrize("what", ["lstm", "lstm bf16", "rnn", "rnn bf16", "rntn"])
def test_too_many_leaves(what, n_good):
    """Every kernel leaves such a batch; the status says so although none of them has latched anything."""
    print("case too many leaves", what, n_good, flush=True)
    if "lstm" in what:
        p = small_params()
    else:
        p = synth.make_rnn_params(5, synth.CELL_RNTN if what == "rntn" else synth.CELL_TREERNN, 50, 16, scale=0.4)
    bad = batch_with_too_many_leaves(n_good)
    assert (bad.n_nodes + bad.n_trees) % 2 == 0 and (bad.left < 0).sum() * 2 == bad.n_nodes + bad.n_trees + 2
    kw = dict(precision=binding.TL_BF16_IN) if "bf16" in what else {}
    for sched in SCHEDULERS:
        run_expect(p, bad, sched, binding.TL_ESTRUCT, **kw)


@pytest.mark.parametrize("make_bad", [lambda: batch_with_too_many_leaves(0), lambda: batch_with_too_many_leaves(40), cyclic_batch, lambda: batch_with_wrong_roots(40, 20, 50)],
                         ids=["three leaves", "three leaves among trees", "cycle", "roots"])
@pytest.mark.parametrize("cell", ["lstm", "rnn", "rntn"])
@pytest.mark.parametrize("keep", [True, False])
def test_backward_of_a_malformed_batch(cell, keep, make_bad):
    """tl_backward returns TL_ESTRUCT (modes -1 and 0), or tl_status does afterwards (mode 1, where the call does not wait)."""
    print("case backward of a malformed batch", cell, keep, flush=True)
    bad = make_bad()
    if cell == "lstm":
        p = small_params()
    else:
        p = synth.make_rnn_params(5, synth.CELL_RNTN if cell == "rntn" else synth.CELL_TREERNN, 50, 16, scale=0.4)
    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        for mode in (0, 1, -1):
            b = net.load(bad)
            binding.tl_set_keep_gates(net.ctx, keep)
            binding.tl_set_async_backward(net.ctx, mode)
            net.forward()                                     # (rejected as well: what it would keep is never read)
            g_h = torch.ones((b["N"], p.hidden), device="cuda")
            code = binding.TL_OK
            try:
                binding.tl_backward(net.ctx, b, g_h, p.embed_dim, rntn=cell == "rntn")
            except binding.TLError as e:
                code = e.code
            if code == binding.TL_OK and mode == 1:
                code = binding.tl_status(net.ctx)
            assert code == binding.TL_ESTRUCT, (mode, binding.tl_strerror(code))
            assert binding.tl_status(net.ctx) == binding.TL_ESTRUCT, mode
    finally:
        net.close()
