"""The fp32 TreeLSTM cells that split their operands into two fp16 terms (data-flow scheduler; leaves of every scheduler),
at the sizes where their tiles, paddings and scales can go wrong.

Tolerance: two terms hold a value to 2^-23 of itself (2^-38 of the largest of its column or row where it is far below that),
a product of two is off by 2^-21 at most, and a sum of at most 1 024 products of order one carries an error of about 1e-6;
2e-5 relative + 2e-6 absolute leaves an order of magnitude (the figures the schedulers are compared with elsewhere)."""
import numpy as np
import pytest
import torch

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
            net.batch["c"].fill_(float("nan"))
            net.forward()
            assert binding.tl_status(net.ctx) == 0
            assert np.array_equal(net.batch["h"].cpu().numpy(), out["h"], equal_nan=True)
        return out
    finally:
        net.close()


def same(a, b, what):
    for key in ("h", "c", "h_root", "c_root"):
        np.testing.assert_allclose(a[key], b[key], rtol=RTOL, atol=ATOL, err_msg="%s %s" % (what, key))
    assert np.array_equal(a["root"], b["root"])


@pytest.mark.parametrize("H,E", [(1, 1), (15, 3), (16, 31), (17, 32), (31, 33), (32, 4), (33, 127), (63, 129), (65, 300), (97, 257),
                                 (129, 385), (193, 513), (301, 99), (449, 641), (511, 1023), (512, 1024)])
def test_sizes_at_the_edges_of_the_tiles(H, E):
    print("case split sizes", H, E, flush=True)
    params = synth.make_treelstm_params(900 + H, 70, E, H, "xavier")
    trees = synth.make_trees(901, [1, 2, 3, 1, 17, 40, 9, 33], ["random", "chain"] * 4, 70)
    got = run(params, trees, "dataflow")
    ref = oracle.forward_params(params, trees, n_threads=8)
    for key in ("h", "c"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)
    same(got, run(params, trees, "ready"), "dataflow / ready")


def test_columns_and_rows_of_very_different_size():
    """Every column of the weights and every embedding row is scaled for itself: sizes from 1e-25 to 1e20 side by side."""
    print("case split scales", flush=True)
    H, E = 48, 40
    p = synth.make_treelstm_params(910, 60, E, H, "xavier")
    rng = np.random.default_rng(1)
    p.u *= (10.0 ** rng.uniform(-25, 0.5, p.u.shape[1])).astype(np.float32)
    p.w_leaf *= (10.0 ** rng.uniform(-3, 0.5, p.w_leaf.shape[1])).astype(np.float32)
    size = 10.0 ** rng.uniform(-25, 1, p.emb.shape[0])
    size[::7] = 1e20                                    # (gates saturate)
    p.emb *= size.astype(np.float32)[:, None]
    trees = synth.make_trees(911, [30, 8, 1, 21], ["random", "chain", "random", "balanced"], 60)
    got = run(p, trees, "dataflow")
    ref = oracle.forward_params(p, trees, n_threads=8)
    for key in ("h", "c"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)


@pytest.mark.parametrize("where", ["u", "w_leaf", "emb"])
def test_infinities_are_summed_in_fp32(where):
    """An infinity has no two terms; its sums are taken from the parameters as given, as with fp32 instructions."""
    print("case split infinity", where, flush=True)
    H, E = 40, 24
    p = synth.make_treelstm_params(920, 30, E, H, "xavier")
    a = getattr(p, where)
    a[3, 5] = np.inf
    trees = synth.make_trees(921, [12, 5, 1, 20], ["random"] * 4, 30)
    with np.errstate(all="ignore"):
        ref = oracle.forward_params(p, trees, n_threads=8)
    got = run(p, trees, "dataflow")
    for key in ("h", "c"):
        assert np.array_equal(np.isnan(got[key]), np.isnan(ref[key])), key
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key, equal_nan=True)


@pytest.mark.parametrize("shape", ["random", "chain"])
def test_slots_whose_lists_do_not_fit_into_lds(shape):
    """More nodes per set of workgroups than the schedule's lists have room for in LDS: they move to the workspace."""
    print("case split large slots", shape, flush=True)
    params = synth.make_treelstm_params(930, 300, 16, 500, "xavier")
    trees = synth.make_trees(931, [1200] * 40, [shape] * 40, 300)
    same(run(params, trees, "dataflow"), run(params, trees, "level_device"), shape)


@pytest.mark.parametrize("first", ["level kernel picked", "rejected"])
@pytest.mark.parametrize("H,E", [(33, 1025), (1, 1025), (47, 1030)])
def test_rows_that_were_internal_nodes_before_become_leaves(H, E, first):
    """The split copy of h outlives a batch.  Rows that a batch marked and nobody wrote (the level kernel was picked; the batch
    was rejected) are leaves in the next one, evaluated by the leaf kernel for long embeddings: with an odd hidden size
    the pad unit beside the last one must read as zero again."""
    print("case split reused rows", H, E, first, flush=True)
    params = synth.make_treelstm_params(940, 40, E, H, "xavier")
    before = synth.make_trees(941, [256] * 3, ["balanced"] * 3, 40)
    if first == "rejected":
        before.word[np.flatnonzero(before.left < 0)[7]] = 40
    after = synth.make_trees(942, [30, 1, 200], ["random", "chain", "random"], 40)       # (no larger in any way: the workspace stays)
    assert ((before.left[:after.n_nodes] >= 0) & (after.left < 0)).sum() > 50
    ref = oracle.forward_params(params, after, n_threads=8)
    net = binding.TreeNet(params, scheduler="dataflow")
    try:
        net.load(before)
        net.forward()
        assert binding.tl_status(net.ctx) == (binding.TL_ESTRUCT if first == "rejected" else binding.TL_OK)
        got = net.run(after)
    finally:
        net.close()
    for key in ("h", "c"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)


def test_leaf_sums_that_overflow_only_when_scaled():
    """6e34 - 3.9e34 - 3.9e34 over three quarters of the embedding row: the first partial sum is beyond the largest number once it is
    scaled by 2^13, the others are not.  The input gate is closed, so c is zero there."""
    print("case split scaled overflow", flush=True)
    H, E = 20, 300
    p = synth.make_treelstm_params(955, 4, E, H, "xavier")
    p.emb[:, 0], p.emb[:, 100], p.emb[:, 200] = 6e34, 3.9e34, 3.9e34
    p.w_leaf[:] = 0
    p.w_leaf[0, 3], p.w_leaf[100, 3], p.w_leaf[200, 3] = 1, -1, -1
    p.b_leaf[2 * H:] = 1
    trees = synth.make_trees(956, [12, 5, 1, 20], ["random"] * 4, 4)
    ref, got = oracle.forward_params(p, trees, n_threads=4), run(p, trees, "dataflow")
    assert (ref["c"][trees.left < 0, 3] == 0).all()
    for key in ("h", "c"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)


@pytest.mark.parametrize("bits", [0xFFFFE000, 0x7FFFE000, 0xFFFFFFFE, 0x7FC00000])
@pytest.mark.parametrize("where", ["b_leaf", "b", "emb"])
def test_a_nan_is_a_result_whatever_its_payload(where, bits):
    """NaNs in neighbouring units whose fp16 halves would be all ones: rows that hold them count as written.  (Only a NaN
    of 32 ones may end a forward with TL_ESTALL.)"""
    print("case split nan", where, hex(bits), flush=True)
    H, E = 34, 20
    p = synth.make_treelstm_params(950, 30, E, H, "xavier")
    a = getattr(p, where)
    at = (slice(4, 8), slice(0, 2)) if where == "emb" else slice(a.shape[0] // H * H - 2 * H + 6, a.shape[0] // H * H - 2 * H + 10)     # output gate
    a.view(np.uint32)[at] = bits
    trees = synth.make_trees(951, [12, 5, 1, 20], ["random"] * 4, 30)
    with np.errstate(all="ignore"):
        ref = oracle.forward_params(p, trees, n_threads=8)
    net = binding.TreeNet(p, scheduler="dataflow", spin_limit=20000)
    try:
        got = net.run(trees)
    finally:
        net.close()
    for key in ("h", "c"):
        assert np.isnan(ref[key]).any() or (where != "emb" and key == "c")
        assert np.array_equal(np.isnan(got[key]), np.isnan(ref[key])), key
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key, equal_nan=True)


def test_batches_beyond_the_range_of_the_split_cell_cost_no_copy_of_h():
    """2^24 nodes and more go to the level scheduler: nothing is allocated for a cell that does not run, results are those of
    the checker, and the next batch in range is evaluated as always."""
    print("case split range", flush=True)
    H, V = 2, 50
    p = synth.make_treelstm_params(960, V, 8, H, "xavier")
    B = (1 << 24) // 3 + 5
    node = np.arange(3 * B, dtype=np.int32)
    root = node % 3 == 0
    trees = synth.TreeBatch(np.arange(0, 3 * B + 1, 3, dtype=np.int32), np.where(root, node + 1, -1).astype(np.int32),
                            np.where(root, node + 2, -1).astype(np.int32), np.where(root, -1, (node * 7) % V).astype(np.int32))
    assert trees.n_nodes >= 1 << 24
    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        net.load(trees)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        net.forward()
        assert binding.tl_status(net.ctx) == 0
        used = free - torch.cuda.mem_get_info()[0]
        # 48 bytes of parents, counters and lists a node; a copy of h would take 128 more, a schedule as many again
        assert used < 64 * trees.n_nodes, used / trees.n_nodes
        some = np.concatenate([np.arange(40), np.arange(B - 40, B)])
        sub, orig = synth.subset(trees, [int(t) for t in some])
        ref = oracle.forward_params(p, sub, n_threads=8)
        for key in ("h", "c"):
            np.testing.assert_allclose(net.batch[key].cpu().numpy()[orig], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)
        small = synth.make_trees(961, [5, 1, 90, 33], ["random"] * 4, V)
        got, ref = net.run(small), oracle.forward_params(p, small, n_threads=8)
        for key in ("h", "c"):
            np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)
    finally:
        net.close()


def test_first_call_on_a_stream_of_its_own():
    """A stream that does not wait for the null stream: what a context clears when it allocates is clear before the call's
    kernels run, also when the workspace grows."""
    print("case split, stream of its own", flush=True)
    H, E = 33, 1025
    p = synth.make_treelstm_params(970, 40, E, H, "xavier")
    batches = [synth.make_trees(971, [30, 7, 1], ["random"] * 3, 40), synth.make_trees(972, [50] * 400, ["random"] * 400, 40)]
    stream = torch.cuda.Stream()
    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        for trees in batches:
            net.load(trees)
            torch.cuda.synchronize()
            net.forward(stream.cuda_stream)
            assert binding.tl_status(net.ctx) == 0
            ref = oracle.forward_params(p, trees, n_threads=8)
            for key in ("h", "c"):
                np.testing.assert_allclose(net.batch[key].cpu().numpy(), ref[key], rtol=RTOL, atol=ATOL, err_msg=key)
    finally:
        net.close()


@pytest.mark.parametrize("H", [35, 64])
def test_few_large_trees_of_either_kind_one_after_the_other(H):
    """Both kernels of the internal nodes are launched for few large trees, the marks are set only for the one that waits
    for them: bushy trees, then deep ones, then bushy ones again through one context."""
    print("case split, few large trees", H, flush=True)
    p = synth.make_treelstm_params(980, 40, 50, H, "xavier")
    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        for i, shape in enumerate(["balanced", "chain", "random", "chain"]):
            trees = synth.make_trees(981 + i, [300, 200, 400], [shape] * 3, 40)
            got, ref = net.run(trees), oracle.forward_params(p, trees, n_threads=8)
            for key in ("h", "c", "h_root", "c_root"):
                np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg="%s %s" % (shape, key))
    finally:
        net.close()


@pytest.mark.parametrize("H,E", [(40, 24), (33, 130), (150, 300)])
def test_forward_after_an_update_is_that_of_a_fresh_context(H, E):
    """tl_sgd_update rebuilds the two terms of U and W_leaf and their scales: afterwards a forward has the bits of a context
    made from the updated parameters, also where a column's largest magnitude has changed.  (Steps of up to 0.05 x 2 a weight:
    gates stay below about 10; the tolerance, 2e-6 for gates of order one, does not hold for the hundreds that larger ones give.)"""
    print("case split update", H, E, flush=True)
    p = synth.make_treelstm_params(990, 60, E, H, "xavier")
    trees = synth.make_trees(991, [30, 8, 1, 21], ["random", "chain", "random", "balanced"], 60)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    grads = dict(d_u=rand(2 * H, 5 * H) * torch.logspace(-4, 0.3, 5 * H, device="cuda"), d_b=rand(5 * H),
                 d_w_leaf=rand(E, 3 * H) * torch.logspace(0.3, -4, 3 * H, device="cuda"), d_b_leaf=rand(3 * H), d_x=rand(trees.n_nodes, E))
    net = binding.TreeNet(p, scheduler="dataflow")
    try:
        before = net.run(trees)
        binding.tl_sgd_update(net.ctx, 0.05, net.batch, grads)
        new = {k: v.cpu().numpy() for k, v in binding.tl_get_params(net.ctx, 60, E, H).items()}
        after = net.run(trees)
    finally:
        net.close()
    assert np.abs(after["h"] - before["h"]).max() > 1e-2
    q = synth.Params(p.cell, 60, E, H, new["emb"], new["w_leaf"], new["b_leaf"], new["u"], new["b"], None)
    fresh = run(q, trees, "dataflow")
    for key in ("h", "c", "h_root", "c_root"):
        assert np.array_equal(after[key], fresh[key]), key
    ref = oracle.forward_params(q, trees, n_threads=8)
    for key in ("h", "c"):
        np.testing.assert_allclose(after[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)


@pytest.mark.parametrize("where", ["u", "w_leaf", "emb", "all"])
def test_entries_of_one_column_or_row_that_differ_by_2_to_the_30(where):
    """Within a column of the weights or a quarter of an embedding row the scale is common: an entry far below the largest one
    keeps an absolute error of 2^-38 of that one.  A gate sums at most 2 H (E) products of such an entry with a
    factor of at most one (3 for an embedding value): 400 x 3 x 2^-38 < 5e-9, far inside the tolerance."""
    print("case split range within", where, flush=True)
    H, E = 96, 200
    p = synth.make_treelstm_params(995, 60, E, H, "xavier")
    rng = np.random.default_rng(6)
    for name in (("u", "w_leaf", "emb") if where == "all" else (where,)):
        a = getattr(p, name)
        a *= (2.0 ** rng.uniform(-30, 0, a.shape)).astype(np.float32) * np.float32(8 if name != "emb" else 3)
    trees = synth.make_trees(996, [30, 8, 1, 21], ["random", "chain", "random", "balanced"], 60)
    got, ref = run(p, trees, "dataflow"), oracle.forward_params(p, trees, n_threads=8)
    for key in ("h", "c"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)


@pytest.mark.parametrize("H,n_trees,leaves,shape", [(48, 90, 9, "random"), (50, 20, 9, "random"), (65, 38, 9, "random"), (65, 39, 9, "random"), (112, 27, 9, "random"),
                                                    (150, 18, 9, "random"), (150, 19, 9, "random"), (150, 37, 70, "chain"), (177, 31, 70, "chain"),
                                                    (250, 24, 70, "chain"), (260, 24, 70, "chain"), (250, 25, 70, "chain")])
def test_slots_inside_one_domain_or_on_all_of_them(H, n_trees, leaves, shape):
    """Both ways of placing the slots, on both sides of the lines between them, with numbers of slots that eight divides and
    that it does not (what is left over lies on all domains): every slot is evaluated once, by all of its column groups."""
    print("case split placement", H, n_trees, leaves, shape, flush=True)
    params = synth.make_treelstm_params(1000 + H, 70, 20, H, "xavier")
    trees = synth.make_trees(1001, [leaves - t % 5 for t in range(n_trees)], [shape] * n_trees, 70)
    got, ref = run(params, trees, "dataflow"), oracle.forward_params(params, trees, n_threads=8)
    for key in ("h", "c", "h_root", "c_root"):
        np.testing.assert_allclose(got[key], ref[key], rtol=RTOL, atol=ATOL, err_msg=key)
