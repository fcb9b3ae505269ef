"""GPU parity of the sweep by layers: steps at their limits (operators, outputs), segments of the plan with a few operators left
over, operators with more outputs and inputs than an entry holds, tensors at the ring's edge, parts of 16 sets, and the graphs
that it must leave to the traversal."""
import numpy as np
import pytest

import graphgen as gg
from helpers import targets_from_sets
from test_gpu_parity import assert_same, oracle_prune
from test_gpu_ring_sweep import draw_targets, prune_words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgn():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_1707_08265_amd as d
    return d


def in_layers(rng, widths, back, out_lo, out_hi, in_max, num_inputs):
    """Operators of layer l read from layers l - back .. l - 1 and the graph's inputs; outputs numbered in order."""
    widths = np.asarray(widths)
    P, start = int(widths.sum()), np.concatenate([[0], np.cumsum(widths)])
    layer = np.repeat(np.arange(widths.size), widths)
    n_out = rng.integers(out_lo, out_hi + 1, P)
    first = num_inputs + np.concatenate([[0], np.cumsum(n_out)])
    fan = np.where(rng.random(P) < 0.02, in_max, rng.integers(0, 4, P))
    op = np.repeat(np.arange(P), fan)
    lo = first[start[np.maximum(layer[op] - np.where(rng.random(op.size) < 0.8, 1, back), 0)]]
    hi = first[start[layer[op]]]
    t = np.where((rng.random(op.size) < 0.05) | (hi <= lo), rng.integers(0, num_inputs, op.size),
                 lo + (rng.random(op.size) * np.maximum(hi - lo, 1)).astype(np.int64))
    i32 = lambda x: x.astype(np.int32)  # noqa: E731
    return gg.Graph(P, int(first[-1]), i32(op), i32(t), i32(np.repeat(np.arange(P), n_out)),
                    i32(num_inputs + np.arange(int(n_out.sum()))), name="layers")


def check(dgn, oracle, g, draws, swept=True, dg=None, buf=None):
    import torch
    dg = dg or dgn.DeviceGraph.from_coo(g)
    for i, tg in enumerate(draws):
        b = buf or dgn.PruneBuffers(dg, tg.num_sets)
        for t in (b.tensor_mask, b.op_mask, b.kept_masks, b.per_query_count, b.kept_count, b.op_flag):
            t.fill_(7)
        b.scratch.fill_(0xAB)
        for call in range(2):
            st = dgn.dgn_stats()
            assert b.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), stats=st) == 0
            assert_same(b.to_host(), oracle_prune(oracle, g, tg)[1], f"draw {i} call {call}")
            assert (st.max_frontier == 0 and st.levels > 0) == swept, (st.levels, st.max_frontier)


WIDTHS = {
    "even": [400] * 60, "step": [512] * 40, "step+1": [513] * 40, "wide": [1700] * 30, "narrow": [41] * 900,
    "ragged": None, "segment": [2048] * 24, "segment+1": [2048] * 24 + [1],
}


@pytest.mark.parametrize("sets", [1, 16, 17, 64])
@pytest.mark.parametrize("widths", list(WIDTHS))
def test_layers(dgn, oracle, widths, sets):
    rng = np.random.default_rng(len(widths) * 100 + sets)
    w = WIDTHS[widths] or rng.integers(1, 1200, 60)
    g = in_layers(rng, w, 4, 1, 2, 3, 50)
    check(dgn, oracle, g, [draw_targets(rng, g, sets, 5)])


@pytest.mark.parametrize("out_lo,out_hi,in_max", [(0, 2, 4), (0, 7, 3), (1, 1, 40), (0, 5, 300), (0, 12, 2)])
def test_operators_with_many_inputs_and_outputs(dgn, oracle, out_lo, out_hi, in_max):
    rng = np.random.default_rng(out_hi * 7 + in_max)
    g = in_layers(rng, rng.integers(200, 700, 50), 3, out_lo, out_hi, in_max, 900)
    check(dgn, oracle, g, [draw_targets(rng, g, q, 9) for q in (3, 40)])


@pytest.mark.parametrize("low,reads,swept", [(1, 40_000, True), (8192, 47_000, True), (8193, 1000, False), (5, 49_153, False)])
def test_how_far_back_and_how_many_graph_inputs(dgn, oracle, low, reads, swept):
    """500 operators to a layer, one output each; every 1 000th operator reads `reads` tensors back."""
    rng = np.random.default_rng(low)
    g = in_layers(rng, [500] * 250, 2, 1, 1, 3, low)
    e = np.flatnonzero((g.in_op % 1000 == 7) & (g.in_op > reads + 500) & (np.diff(g.in_op, prepend=-1) > 0))
    g.in_tensor[e] = low + g.in_op[e] - reads
    check(dgn, oracle, g, [draw_targets(rng, g, 20, 4)], swept)


def test_targets_at_the_ends_and_none(dgn, oracle):
    rng = np.random.default_rng(5)
    g = in_layers(rng, [300] * 70, 3, 1, 2, 3, 20)
    T = g.num_tensors
    draws = [targets_from_sets(s, 3) for s in ([[T - 1], [0], [T - 1, T - 1, 20]], [[], [], []], [[3], [19], []], [[T // 2], [T // 2 + 1], [40]])]
    check(dgn, oracle, g, draws)
    many = gg.targets_range(3, 64, 900, 1000, 0, T)                      # 60 000 targets: in every step
    check(dgn, oracle, g, [many])


def test_bad_targets_and_other_buffers_contents(dgn, oracle):
    """A target out of range is an error, and the next call is right; sweep, wide levels and one launch per level in the same buffers."""
    import torch
    rng = np.random.default_rng(6)
    g = in_layers(rng, [350] * 80, 3, 1, 2, 3, 20)
    dg = dgn.DeviceGraph.from_coo(g)
    tg = draw_targets(rng, g, 30, 4)
    ref = oracle_prune(oracle, g, tg)[1]
    buf = dgn.PruneBuffers(dg, 30)
    ptr, idx = torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda()
    bad = idx.clone()
    bad[0] = g.num_tensors
    seen = []
    for knobs, targets in (({}, idx), ({}, idx), ({}, idx), ({}, bad), ({}, idx), ({"traversal": 2}, idx), ({"traversal": 2}, idx), ({}, idx), ({}, idx),
                           ({"traversal": 1}, idx)):
        st = dgn.dgn_stats()
        rc = buf.prune(ptr, targets, options=dgn.dgn_options(recycle=1, **knobs), stats=st)
        assert rc == (dgn.DGN_ERR_ID_OUT_OF_RANGE if targets is bad else 0)
        seen.append(int(st.recycled))
        if rc == 0:
            assert_same(buf.to_host(), ref, str(knobs))
    # (the buffers' first call leaves nothing to recognise, nor does an error or the other way's result)
    assert seen == [0, 0, 1, 1, 0, 0, 1, 0, 1, 0], seen


@pytest.mark.parametrize("make", [lambda: gg.rnn(300, 80, 5), lambda: gg.powerlaw(60_000, 5), lambda: gg.layered(40_000, 5)])
def test_chains_and_reads_from_all_over_are_traversed(dgn, oracle, make):
    import torch
    g = make()
    tg = draw_targets(np.random.default_rng(3), g, 5, 2)
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), 5)
    st = dgn.dgn_stats()
    assert buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), stats=st) == 0
    assert_same(buf.to_host(), oracle_prune(oracle, g, tg)[1], "traversed")
    assert st.max_frontier > 0


def test_layers_in_which_operators_read_each_other(dgn, oracle):
    """It looks like layers where it is sampled, but most operators read the one before: left to the traversal, now and later."""
    rng = np.random.default_rng(8)
    g = in_layers(rng, [400] * 60, 3, 1, 1, 3, 20)
    e = np.flatnonzero((np.diff(g.in_op, append=-1) != 0) & (np.diff(g.in_op, prepend=-1) == 0))      # last of several inputs
    g.in_tensor[e] = 20 + g.in_op[e] - 1
    check(dgn, oracle, g, [draw_targets(rng, g, 8, 3)], swept=False)


# With more targets than the sweep holds, a step takes half as long again (the measurements stand beside the rule in api.hip): few sets on
# many operators are left to the levels, and so are the words of a call with so many targets on the largest graphs.
@pytest.mark.parametrize("layers,width,sets,targets,swept", [
    (200, 500, 5, 2000, True), (200, 600, 5, 3000, False), (100, 500, 1, 3000, True), (100, 600, 1, 3000, False), (200, 600, 16, 3000, True),
    (1000, 210, 8, 3000, True), (300, 700, 8, 3000, False), (500, 700, 64, 3000, False), (500, 700, 64, 1500, True)])
def test_more_targets_than_the_sweep_holds(dgn, oracle, layers, width, sets, targets, swept):
    rng = np.random.default_rng(layers + sets)
    g = in_layers(rng, [width] * layers, 3, 1, 2, 3, 50)
    cuts = np.sort(rng.integers(0, targets + 1, sets - 1))
    tg = targets_from_sets([[int(t) for t in part] for part in np.split(rng.integers(0, g.num_tensors, targets), cuts)], sets)
    check(dgn, oracle, g, [tg], swept)


@pytest.mark.parametrize("sets,per_set,launches", [(150, 5, 3 * 5), (150, 20, None), (69, 3, 2 * 5), (66, 3, None)])
def test_words_of_sets_on_many_layers(dgn, oracle, sets, per_set, launches):
    """Each word is swept by itself, five launches; with 3 000 targets in all, of which a word might own most, on 350 000 operators none
    is, nor a last word of two sets."""
    rng = np.random.default_rng(per_set)
    g = in_layers(rng, [700] * 500, 3, 1, 2, 3, 50)
    tg = targets_from_sets([[int(t) for t in rng.integers(0, g.num_tensors, per_set)] for _ in range(sets)], 64)
    took = prune_words(dgn, oracle, g, tg, sets)
    assert took == launches if launches else took > 6 * -(-sets // 64)


@pytest.mark.parametrize("layers,width,sets,swept", [(200, 1000, 4, True), (201, 1000, 4, False), (201, 1000, 5, True), (201, 1000, 63, True),
                                                     (1000, 201, 1, True), (1000, 300, 1, True), (1000, 301, 1, False), (1000, 301, 5, True)])
def test_few_sets_on_many_operators(dgn, oracle, layers, width, sets, swept):
    rng = np.random.default_rng(layers + sets)
    g = in_layers(rng, [width] * layers, 3, 1, 2, 3, 50)
    check(dgn, oracle, g, [draw_targets(rng, g, sets, 9)], swept)


@pytest.mark.parametrize("sets", [1, 16, 64])
@pytest.mark.parametrize("targets", [512, 513, 1025, 1537, 2047, 2048, 2049, 3000])
def test_targets_of_one_workgroup(dgn, oracle, targets, sets):
    """All of a call's targets in one set, or spread unevenly over 16 (one workgroup's) or 64: a thread holds one to four of them; 2 049
    go by way of M.  And with a bad one among them."""
    import torch
    rng = np.random.default_rng(targets + sets)
    g = in_layers(rng, [300] * 70, 3, 1, 2, 3, 20)
    cuts = np.sort(rng.integers(0, targets + 1, sets - 1))
    tg = targets_from_sets([[int(t) for t in part] for part in np.split(rng.integers(0, g.num_tensors, targets), cuts)], sets)
    dg, buf = dgn.DeviceGraph.from_coo(g), None
    check(dgn, oracle, g, [tg], dg=dg)
    buf = dgn.PruneBuffers(dg, sets)
    for place, bad in ((0, -1), (targets - 1, g.num_tensors), (targets // 2, 2**31 - 1)):
        wrong = tg.tgt_idx.copy()
        wrong[place] = bad
        assert buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(wrong).cuda()) == dgn.DGN_ERR_ID_OUT_OF_RANGE
        check(dgn, oracle, g, [tg], dg=dg, buf=buf)


@pytest.mark.parametrize("flags", ["none", "unaligned", "ragged", "whole"])
def test_backward_prune_with_flag_bytes_of_its_own(dgn, oracle, flags):
    """The first stage of a backward prune keeps flag bytes in its scratch where the caller's cannot be cleared in whole words (then one more
    launch clears them): no op_flag, one at an odd address, a number of operators that is no multiple of 8."""
    import torch
    rng = np.random.default_rng(len(flags))
    g = in_layers(rng, [300] * 70 + ([5] if flags == "ragged" else []), 3, 1, 2, 3, 20)
    obj = rng.integers(0, 20, 50).astype(np.int32)
    wrt = rng.integers(g.num_tensors - 600, g.num_tensors, 50).astype(np.int32)
    ref = oracle.backward_prune(oracle.build_adjacency(g.num_ops, g.num_tensors, g.in_op, g.in_tensor, g.out_op, g.out_tensor), obj, wrt)
    buf = dgn.BackwardPruneBuffers(dgn.DeviceGraph.from_coo(g), 64)
    big = torch.full((g.num_ops + 16,), 77, dtype=torch.uint8, device="cuda")
    if flags != "ragged":
        buf.op_flag = {"none": None, "unaligned": big[3:3 + g.num_ops], "whole": big[8:8 + g.num_ops]}[flags]
    for call in range(3):                                    # (the last one with recycled buffers)
        st = dgn.dgn_stats()
        assert buf.backward_prune(torch.from_numpy(obj).cuda(), torch.from_numpy(wrt).cuda(), stats=st) == 0
        assert st.max_frontier == 0 and st.launches == (5 if flags == "whole" else 6)
        own, buf.op_flag = buf.op_flag, buf.op_flag if buf.op_flag is not None else torch.zeros_like(big[:g.num_ops])
        out = buf.to_host()
        buf.op_flag = own
        for name in ("tensor_mask", "op_mask", "kept_ops", "kept_masks", "kept_count", "per_query_count") + (("op_flag",) if own is not None else ()):
            assert np.array_equal(out[name], getattr(ref, name)), (name, call)
    if flags in ("unaligned", "whole"):
        assert int((big == 77).sum()) == 16                  # nothing written outside


@pytest.mark.parametrize("layers,reads,swept", [(60, 20, False), (60, 30, True), (330, 30, False), (6, 7, True)])
def test_short_steps(dgn, oracle, layers, reads, swept):
    """Layers of 400 in which every operator also reads the tensor `reads` before its own, where no sample is taken: steps of so many.  More
    than 64 steps of fewer than 24 operators, or more than 4 096 steps, are left to the traversal, now and later."""
    rng = np.random.default_rng(reads)
    g = in_layers(rng, [400] * layers, 3, 1, 1, 3, 20)
    ops = np.arange(reads, g.num_ops, dtype=np.int32) if reads > 7 else np.arange(g.num_ops - 200, g.num_ops, dtype=np.int32)
    op, t = np.concatenate([g.in_op, ops]), np.concatenate([g.in_tensor, (20 + ops - reads).astype(np.int32)])
    order = np.argsort(op, kind="stable")                    # (behind the operator's other inputs)
    g = gg.Graph(g.num_ops, g.num_tensors, op[order].astype(np.int32), t[order].astype(np.int32), g.out_op, g.out_tensor, name="short steps")
    check(dgn, oracle, g, [draw_targets(rng, g, 8, 3)], swept)


def test_an_incremental_call_between_swept_ones(dgn, oracle):
    """It has levels, and leaves nothing that the next call recognises."""
    import torch
    rng = np.random.default_rng(9)
    g = in_layers(rng, [350] * 80, 3, 1, 2, 3, 20)
    dg, buf = dgn.DeviceGraph.from_coo(g), None
    sets = [[[int(t) for t in rng.integers(0, g.num_tensors, 3)] for _ in range(30)] for _ in range(2)]
    first, added, both = [targets_from_sets(s, 30) for s in (sets[0], sets[1], [a + b for a, b in zip(*sets)])]
    buf = dgn.PruneBuffers(dg, 30)
    seen = []
    for tg, ref, knobs in ((first, first, {}), (first, first, {}), (added, both, {"incremental": 1}), (first, first, {}), (first, first, {}),
                           (added, both, {"incremental": 1}), (added, added, {"traversal": 2}), (added, added, {})):
        st = dgn.dgn_stats()
        rc = buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), options=dgn.dgn_options(**knobs), stats=st)
        assert rc == 0 and (st.max_frontier == 0) == (not knobs)
        assert_same(buf.to_host(), oracle_prune(oracle, g, ref)[1], str(knobs))
        seen.append(int(st.recycled))
    assert seen == [0, 0, 0, 0, 1, 0, 0, 0], seen
