"""GPU parity of the ring sweep (graphs whose tensors are numbered as they are created and that read recent tensors or
graph inputs only): sizes at the edges of words, groups and the ring, operators with more outputs and inputs than a
lane keeps in registers, graphs without operators, more targets than fit in LDS, recycled buffers."""
import numpy as np
import pytest

import graphgen as gg
from helpers import targets_from_sets
from test_gpu_parity import assert_same, oracle_prune

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgn():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_1707_08265_amd as d
    return d


def recorded(rng, num_graphs, ops, window, out_max, in_max, num_inputs, empty_every=0):
    """Packed graphs of 1..ops operators (exactly `ops` for a single graph), outputs 0..out_max numbered in order, inputs
    from the last `window` tensors or the graph's inputs; every empty_every-th graph has tensors and no operator."""
    op_off, t_off, io, it, oo, ot = [0], [0], [], [], [], []
    for gi in range(num_graphs):
        P = ops if num_graphs == 1 else int(rng.integers(1, ops + 1))
        if empty_every and gi % empty_every == 0:
            P = 0
        lo = t_off[-1]
        n_out = rng.integers(0 if out_max > 2 else 1, out_max + 1, P)
        first = lo + num_inputs + np.cumsum(n_out) - n_out
        fan = rng.integers(0, in_max + 1, P)
        op = np.repeat(np.arange(P), fan)
        back = rng.integers(1, window + 1, op.size)
        t = np.where(rng.random(op.size) < 0.2, lo + rng.integers(0, num_inputs, op.size), np.maximum(first[op] - back, lo))
        io.append(op_off[-1] + op)
        it.append(t)
        oo.append(op_off[-1] + np.repeat(np.arange(P), n_out))
        ot.append(lo + num_inputs + np.arange(n_out.sum()))
        op_off.append(op_off[-1] + P)
        t_off.append(lo + num_inputs + int(n_out.sum()))
    cat = lambda xs: np.concatenate(xs).astype(np.int32)  # noqa: E731
    many = num_graphs > 1
    return gg.Graph(op_off[-1], t_off[-1], cat(io), cat(it), cat(oo), cat(ot), num_graphs,
                    np.asarray(op_off, np.int64) if many else None, np.asarray(t_off, np.int64) if many else None, "recorded")


def draw_targets(rng, g, Q, most):
    off = g.graph_tensor_offsets if g.num_graphs > 1 else [0, g.num_tensors]
    sets = []
    for gi in range(g.num_graphs):
        lo, hi = int(off[gi]), int(off[gi + 1])
        sets += [[int(t) for t in rng.integers(lo, hi, int(rng.integers(0, most + 1)))] for _ in range(Q)]
    return targets_from_sets(sets, Q)


def check(dgn, oracle, g, draws, swept=True):
    import torch
    dg = dgn.DeviceGraph.from_coo(g)
    buf = dgn.PruneBuffers(dg, draws[0].num_sets)
    for t in (buf.tensor_mask, buf.op_mask, buf.kept_masks, buf.per_query_count, buf.kept_count):
        t.fill_(-1)
    buf.op_flag.fill_(7)
    for i, tg in enumerate(draws):
        st = dgn.dgn_stats()
        rc = buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), stats=st)
        assert rc == 0, dgn.dgn_strerror(rc)
        assert not swept or st.launches <= 3                             # the sweep and the ordered list, no levels
        assert_same(buf.to_host(), oracle_prune(oracle, g, tg)[1], f"call {i}")


# (graphs, operators, window, most outputs, most inputs, graph inputs): one wave, four waves and sixteen waves per graph
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 1, 3, 1), (1, 64, 1, 1, 1, 4), (1, 65, 3, 2, 3, 4), (1, 256, 40, 2, 4, 16), (1, 257, 64, 2, 3, 16),
    (1, 1023, 1, 1, 2, 2), (1, 1025, 90, 2, 4, 16), (1, 4097, 700, 5, 7, 30), (1, 16384, 64, 2, 3, 16),
    (1, 16385, 64, 2, 3, 16), (3, 2000, 50, 2, 3, 16), (70, 300, 64, 2, 3, 16), (300, 200, 30, 3, 6, 5), (2100, 90, 64, 4, 5, 16)])
def test_shapes(dgn, oracle, shape):
    G, P, window, out_max, in_max, low = shape
    rng = np.random.default_rng(P * 7 + G)
    g = recorded(rng, G, P, window, out_max, in_max, low, empty_every=9 if G > 9 else 0)
    Q = 64 if P % 2 else 5
    check(dgn, oracle, g, [draw_targets(rng, g, Q, 3) for _ in range(4)])


# Graphs read at most 64 tensors back are swept in segments (two launches, or one where the whole graph is one segment):
# sizes at the edges of words and segments, operators without outputs and with many, more graph inputs than a wave has lanes, the
# reach that is just too far, batches with short and empty graphs, targets that go through the masks.
@pytest.mark.parametrize("shape,segments", [
    ((1, 448, 64, 2, 3, 16), False), ((1, 449, 64, 2, 3, 16), True), ((1, 1024, 64, 2, 3, 1), True), ((1, 1025, 64, 2, 3, 16), True),
    ((1, 1153, 1, 1, 1, 1), True), ((1, 2049, 64, 6, 7, 100), True), ((1, 3000, 64, 3, 3, 300), True), ((1, 3000, 65, 2, 3, 16), False),
    ((1, 16321, 30, 1, 2, 5), True), ((1, 20000, 64, 4, 5, 70), True), ((3, 900, 64, 2, 3, 16), None), ((6, 5000, 64, 3, 4, 80), None),
    ((90, 2500, 64, 2, 3, 16), None), ((260, 4000, 64, 2, 3, 16), None)])
@pytest.mark.parametrize("Q,most", [(1, 3), (64, 2), (64, 200)])
def test_segments(dgn, oracle, shape, segments, Q, most):
    import torch
    G, P, window, out_max, in_max, low = shape
    rng = np.random.default_rng(P * 11 + G + Q + most)
    g = recorded(rng, G, P, window, out_max, in_max, low, empty_every=9 if G > 9 else 0)
    draws = [draw_targets(rng, g, Q, most if G < 9 else min(most, 40)) for _ in range(2)]
    check(dgn, oracle, g, draws + draws[:1])
    if segments is None:
        return
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), Q)
    st = dgn.dgn_stats()
    assert buf.prune(torch.from_numpy(draws[0].tgt_rowptr).cuda(), torch.from_numpy(draws[0].tgt_idx).cuda(), stats=st) == 0
    assert st.launches == (2 if segments or P > 16384 else 1) and st.levels > 0


@pytest.mark.parametrize("G,ops,segments", [(20, 5000, True), (40, 2500, True), (5, 400, False)])
def test_batches_in_segments(dgn, oracle, G, ops, segments):
    """Settling steps are added up over all segments' sweeps of all graphs, six for every word here; in one piece they are the largest
    graph's alone, one for every word of all."""
    import torch
    rng = np.random.default_rng(G + ops)
    g = recorded(rng, G, ops, 64, 2, 3, 16)
    tg = draw_targets(rng, g, 64, 2)
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), 64)
    st = dgn.dgn_stats()
    assert buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), stats=st) == 0
    assert_same(buf.to_host(), oracle_prune(oracle, g, tg)[1], "batch")
    words = -(-np.diff(np.asarray(g.graph_op_offsets)) // 64)
    print(f"{G} graphs of up to {ops}: {int(st.levels)} settling steps, {int(words.sum())} words, the largest {int(words.max())}", flush=True)
    assert (st.levels > 3 * words.sum()) == segments


# Targets are looked for in rows of 64, four rows at a time, by one wave of a segment or eight (batches: (260, 2000) is the one wave's);
# 2 048 fit in LDS, more go through the masks.
@pytest.mark.parametrize("G,ops", [(1, 460), (1, 5000), (6, 1500), (260, 2000)])
@pytest.mark.parametrize("targets", [1, 64, 65, 257, 2047, 2048, 2049, 5000])
def test_segments_and_the_number_of_targets(dgn, oracle, G, ops, targets):
    """All in one set of each graph, or spread over 64 unevenly with empty ones among them; a bad one among them is an error."""
    import torch
    rng = np.random.default_rng(G + ops + targets)
    g = recorded(rng, G, ops, 64, 2, 3, 16)
    off = np.array([0, g.num_tensors]) if G == 1 else np.asarray(g.graph_tensor_offsets)
    for sets in (1, 64):
        lists = []
        for lo, hi in zip(off, off[1:]):
            t = rng.integers(lo, hi, targets)
            cuts = np.sort(rng.integers(0, targets + 1, sets - 1)) if sets > 1 else []
            lists += [[int(x) for x in part] for part in np.split(t, cuts)]
        check(dgn, oracle, g, [targets_from_sets(lists, sets)], G < 64)
    bad = targets_from_sets(lists, sets)
    bad.tgt_idx[-1] = g.num_tensors
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), sets)
    assert buf.prune(torch.from_numpy(bad.tgt_rowptr).cuda(), torch.from_numpy(bad.tgt_idx).cuda()) == dgn.DGN_ERR_ID_OUT_OF_RANGE


@pytest.mark.parametrize("G,ops", [(1, 800), (8, 800)])
def test_many_targets_cost_no_multiple_of_a_prune(dgn, G, ops):
    """32 000 targets of a graph against 64, both in segments: a little over twice as long; looked at one after the other by the one
    wave of each segment they took ten times and more."""
    import time
    import torch
    rng = np.random.default_rng(G)
    g = recorded(rng, G, ops, 64, 2, 3, 16)
    off = np.array([0, g.num_tensors]) if G == 1 else np.asarray(g.graph_tensor_offsets)
    dg, took = dgn.DeviceGraph.from_coo(g), []
    for per_set in (1, 500):
        idx = np.concatenate([rng.integers(lo, hi, 64 * per_set) for lo, hi in zip(off, off[1:])]).astype(np.int32)
        ptr = np.arange(0, 64 * G + 1, dtype=np.int32) * per_set
        buf, ptr, idx = dgn.PruneBuffers(dg, 64), torch.from_numpy(ptr).cuda(), torch.from_numpy(idx).cuda()
        best = 1.0
        for _ in range(20):
            t = time.perf_counter()
            assert buf.prune(ptr, idx) == 0
            best = min(best, time.perf_counter() - t)
        took.append(best)
    assert took[1] < 5 * took[0], took


@pytest.mark.parametrize("G", [1, 100])
def test_more_targets_than_fit_in_lds_go_through_the_masks(dgn, oracle, G):
    rng = np.random.default_rng(G)
    g = recorded(rng, G, 3000 if G == 1 else 400, 64, 2, 3, 16)
    draws = [draw_targets(rng, g, 64, 100), draw_targets(rng, g, 64, 1)]
    if G > 1:                                                            # one graph with far more than the others
        few = draw_targets(rng, g, 64, 1)
        n = np.diff(few.tgt_rowptr)
        sets = [list(few.tgt_idx[a:a + k]) for a, k in zip(few.tgt_rowptr, n)]
        lo, hi = int(g.graph_tensor_offsets[7]), int(g.graph_tensor_offsets[8])
        sets[7 * 64 + 3] = [int(t) for t in rng.integers(lo, hi, 900)]
        draws.append(targets_from_sets(sets, 64))
    check(dgn, oracle, g, draws + draws[:1])


# (operators, most outputs, sets, most targets per set): a ragged last word, words without targets, one operator, more
# words than the scratch buffer has room for at once (hardly any tensors), targets that go through the masks
@pytest.mark.parametrize("shape", [(3001, 2, 150, 4), (20000, 2, 129, 2), (1, 1, 65, 1), (9000, 0, 20000, 1), (700, 3, 640, 90)])
def test_words_of_sets(dgn, oracle, shape):
    P, out_max, sets, most = shape
    rng = np.random.default_rng(P + sets)
    g = recorded(rng, 1, P, 64, max(out_max, 1), 3, 16)
    if out_max == 0:                                                     # operators that write nothing, but for one
        keep = g.out_op == P // 2
        g = gg.Graph(P, 17, g.in_op, g.in_tensor % 16, g.out_op[keep], np.full(int(keep.sum()), 16, np.int32))
    tg = targets_from_sets([[int(t) for t in rng.integers(0, g.num_tensors, int(rng.integers(0, most + 1)))]
                            for _ in range(sets)], 64)
    launches = prune_words(dgn, oracle, g, tg, sets)
    assert launches <= 2 * -(-sets // 6400)                              # two for a hundred words at once, at least


def prune_words(dgn, oracle, g, tg, sets, flags=True, code=0, good=None):
    """One call of dgn_prune_words, every word (or the first `good`) against the oracle; how many kernels it launched."""
    import torch
    W, P, T = (sets + 63) // 64, g.num_ops, g.num_tensors
    dg = dgn.DeviceGraph.from_coo(g)
    new = lambda n, t: torch.full((W, n), -1 if t != torch.uint8 else 7, dtype=t, device="cuda")  # noqa: E731
    out = {"tensor_mask": new(T, torch.int64), "op_mask": new(P, torch.int64), "op_flag": new(P, torch.uint8) if flags else None,
           "kept_ops": new(P, torch.int32), "kept_masks": new(P, torch.int64), "kept_count": new(1, torch.int64),
           "per_query_count": new(64, torch.int64)}
    rc, nbytes = dgn.dgn_prune_workspace(dg.handle, 64)
    scratch = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    ptr, idx = torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda()
    st = dgn.dgn_stats()
    rc = dgn.dgn_prune_words(dg.handle, sets, idx.numel(), ptr, idx, *out.values(), scratch, nbytes, stats=st)
    assert rc == code, dgn.dgn_strerror(rc)
    host = {k: v.cpu().numpy() for k, v in out.items() if v is not None}
    for w in range(W if good is None else good):
        rows = tg.tgt_rowptr[64 * w:64 * w + 65]
        one = targets_from_sets([list(tg.tgt_idx[a:b]) for a, b in zip(rows, rows[1:])], 64)
        ref = oracle_prune(oracle, g, one)[1]
        n = int(host["kept_count"][w, 0])
        assert n == int(ref.kept_count[0])
        for name in ("tensor_mask", "op_mask", "per_query_count") + (("op_flag",) if flags else ()):
            assert np.array_equal(host[name][w].view(getattr(ref, name).dtype)[:getattr(ref, name).size], getattr(ref, name)), (name, w)
        assert np.array_equal(host["kept_ops"][w, :n], ref.kept_ops[:n])
        assert np.array_equal(host["kept_masks"][w, :n].view(np.uint64), ref.kept_masks[:n])
    return int(st.launches)


@pytest.mark.parametrize("flags", [True, False])
def test_words_of_sets_with_a_single_word_left_over(dgn, oracle, flags):
    """One word more than the scratch buffer has room for at once, no whole number of 8-byte words of flags: the last word is
    swept alone in the layout for many, which has no place for flag bytes (see test_scratch_layout.py)."""
    P = 20001
    rng = np.random.default_rng(P)
    g = recorded(rng, 1, P, 64, 2, 3, 16)
    dg = dgn.DeviceGraph.from_coo(g)
    _, nbytes = dgn.dgn_prune_workspace(dg.handle, 64)
    log = 512 + 64 * 64 + 64 * 4 * max(4096, g.num_tensors // 256)       # the header and the log come first
    at_once = (nbytes - log - 768) // ((P // 64 + 2) * 12 + 16)
    assert at_once > 100
    for words, launches in ((at_once, 2), (at_once + 1, 4)):
        sets = 64 * words - 5
        tg = targets_from_sets([[int(rng.integers(0, g.num_tensors))] for _ in range(sets)], 64)
        assert prune_words(dgn, oracle, g, tg, sets, flags) == launches


@pytest.mark.parametrize("recorded_order", [True, False])
def test_words_before_a_bad_target_are_complete(dgn, oracle, recorded_order):
    rng = np.random.default_rng(6)
    g = recorded(rng, 1, 2000, 64, 2, 3, 16)
    if not recorded_order:                                               # (word by word then)
        g = gg.Graph(g.num_ops, g.num_tensors + 1, g.in_op, g.in_tensor, g.out_op, g.out_tensor)
    sets = [[int(t) for t in rng.integers(0, g.num_tensors, 2)] for _ in range(64 * 4)]
    sets[64 * 2 + 5][1] = g.num_tensors + 3
    prune_words(dgn, oracle, g, targets_from_sets(sets, 64), len(sets), code=dgn.DGN_ERR_ID_OUT_OF_RANGE, good=2)


def test_graphs_that_the_ring_cannot_hold_take_another_path(dgn, oracle):
    """Tensor ids out of order, an unread tensor behind the last output, an input further back than LDS is large."""
    import torch
    rng = np.random.default_rng(3)
    g = recorded(rng, 1, 3000, 64, 2, 3, 16)
    tg = draw_targets(rng, g, 64, 2)
    g2, tg2, _ = gg.relabel_tensors(g, tg, 5)
    g3 = gg.Graph(g.num_ops, g.num_tensors + 1, g.in_op, g.in_tensor, g.out_op, g.out_tensor)
    far = recorded(rng, 1, 30000, 64, 2, 3, 16)
    far.in_tensor[-1] = far.out_tensor[0]
    for h, t in ((g2, tg2), (g3, tg), (far, draw_targets(rng, far, 64, 2))):
        dg = dgn.DeviceGraph.from_coo(h)
        buf = dgn.PruneBuffers(dg, 64)
        st = dgn.dgn_stats()
        assert buf.prune(torch.from_numpy(t.tgt_rowptr).cuda(), torch.from_numpy(t.tgt_idx).cuda(), stats=st) == 0
        assert st.launches > 3
        assert_same(buf.to_host(), oracle_prune(oracle, h, t)[1], "another path")


@pytest.mark.parametrize("G", [1, 8])
def test_a_caller_that_asks_for_the_level_trace_gets_it(dgn, oracle, G):
    """The sweep has no levels: with a trace buffer the same graphs are traversed level by level."""
    import torch
    rng = np.random.default_rng(G)
    g = recorded(rng, G, 2000, 64, 2, 3, 16)
    tg = draw_targets(rng, g, 7, 3)
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), 7)
    ptr, idx = torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda()
    trace = np.full((4096, 4), -77, np.int32)
    for call in range(4):                                                # in turn with calls that are swept
        st = dgn.dgn_stats()
        if call % 2:
            st.level_trace, st.level_trace_cap = trace.ctypes.data, trace.shape[0]
        assert buf.prune(ptr, idx, stats=st) == 0
        assert (st.launches > 3) == bool(call % 2)
        assert_same(buf.to_host(), oracle_prune(oracle, g, tg)[1], f"call {call}")
        if call % 2:
            rows = trace[:int(st.levels)]
            assert 0 < len(rows) < 4096 and (rows[:, 0] >= 0).all() and (rows[:, 1] >= 0).all() and (trace[len(rows):] == -77).all()
            assert rows[:, 0].max() == st.max_frontier > 0 and st.atomic_updates > 0
            trace.fill(-77)


@pytest.mark.parametrize("G,ops", [(1, 2000), (1, 20000), (8, 2000), (100, 500)])
def test_phase_times_of_a_sweep(dgn, G, ops):
    """profile = 1: the kernels behind the sweep are phases of their own, and all phases add up; profile = 2: the sweep alone."""
    import torch
    rng = np.random.default_rng(G + ops)
    g = recorded(rng, G, ops, 64, 2, 3, 16)
    tg = draw_targets(rng, g, 7, 3)
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), 7)
    ptr, idx = torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda()
    for profile in (1, 2):
        st = dgn.dgn_stats()
        assert buf.prune(ptr, idx, options=dgn.dgn_options(profile=profile), stats=st) == 0
        ms = list(st.phase_ms)
        assert st.launches <= 3 and ms[2] > 0                            # DGN_PHASE_TRAVERSE
        if profile == 2:
            assert [m for i, m in enumerate(ms) if i != 2 and m != 0] == []
        else:
            assert ms[1] == ms[3] == 0 and (ms[5] > 0 or st.launches == 1) and (ms[4] > 0 or G == 1)
            assert abs(sum(ms[:6]) - ms[6]) < 0.01 + 0.02 * ms[6]


# Which single graphs are swept (the measurements stand beside the rule in api.hip): there is room for four waves and what the
# operators read (35 layers of 324: for one only), and few operators if they read from all over; beyond 16 384 operators
# only where everything is read at once, and few where chains may die out; more with several words of sets.
@pytest.mark.parametrize("family,size,words,swept", [
    ("cnn", (80, 150), 1, True), ("cnn", (33, 255), 1, True), ("cnn", (20, 400), 1, True), ("cnn", (35, 324), 1, False),
    ("powerlaw", (4000,), 1, True), ("powerlaw", (4200,), 1, False), ("powerlaw", (6000,), 2, True), ("cnn", (200, 90), 1, False), ("layered", (20000,), 1, True),
    ("rnn", (200, 80), 1, True), ("rnn", (300, 80), 1, False), ("rnn", (300, 80), 2, True), ("rnn", (700, 80), 2, False),
    ("rnn", (1500, 80), 1, False)])
def test_which_single_graphs_are_swept(dgn, oracle, family, size, words, swept):
    import torch
    g = gg.cnn(*size, 5)[0] if family == "cnn" else getattr(gg, family)(*size, 5)
    tg = gg.targets_range(3, 64 * words, 1, 3, 16, g.num_tensors)
    if words > 1:
        launches = prune_words(dgn, oracle, g, tg, 64 * words)
    else:
        buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), 64)
        st = dgn.dgn_stats()
        assert buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), stats=st) == 0
        assert_same(buf.to_host(), oracle_prune(oracle, g, tg)[1], "single word")
        launches = st.launches
    assert (launches <= 2) == swept, launches


@pytest.mark.parametrize("family,size,swept", [("layered", (30000,), True), ("batch", (4, 25000), True), ("rnn", (400, 80), False)])
def test_long_thin_graphs_are_swept_once_a_prune_has_shown_their_chains(dgn, oracle, family, size, swept):
    import torch
    g = gg.batch_layered(*size, 5)[0] if family == "batch" else getattr(gg, family)(*size, 5)
    tg = draw_targets(np.random.default_rng(3), g, 9, 2)
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), 9)
    ref = oracle_prune(oracle, g, tg)[1]
    for call in range(3):
        st = dgn.dgn_stats()
        assert buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(), stats=st) == 0
        assert_same(buf.to_host(), ref, f"call {call}")
        assert (st.launches <= 3) == (swept and call > 0), (call, st.launches)


@pytest.mark.parametrize("count,last", [(2701, 64), (2700, 64), (2703, 128), (2701, 63), (2701, 65)])
def test_wide_operators_at_the_very_end_of_a_large_batch(dgn, oracle, count, last):
    """So many operators that a wave of the build walks more than 64 of them, and the widest 64 of all are the last ones, which
    mostly begin in one step of a wave and end in its next: the ring has to hold their outputs."""
    rng = np.random.default_rng(count + last)
    P = np.append(np.full(count, 200), last)
    op_off = np.concatenate([[0], np.cumsum(P)])
    n_out = np.ones(op_off[-1], np.int64)
    n_out[-last:] = np.where(np.arange(last) < last - 64, 1, 40)
    graph = np.repeat(np.arange(count + 1), P)
    t_off = np.concatenate([[0], np.cumsum(4 + np.add.reduceat(n_out, op_off[:-1]))])
    first = 4 * (graph + 1) + np.cumsum(n_out) - n_out
    op, out_op = np.arange(op_off[-1]), np.repeat(np.arange(op_off[-1]), n_out)
    in_op = np.repeat(op, 2)
    in_t = np.maximum(first[in_op] - rng.integers(1, 9, in_op.size), t_off[graph[in_op]])
    out_t = 4 * (graph[out_op] + 1) + np.arange(out_op.size)
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    g = gg.Graph(int(op_off[-1]), int(t_off[-1]), i32(in_op), i32(in_t), i32(out_op), i32(out_t), count + 1, op_off.astype(np.int64),
                 t_off.astype(np.int64), "wide end")
    check(dgn, oracle, g, [draw_targets(rng, g, 3, 2)])


@pytest.mark.parametrize("shuffled", ["", "inputs", "outputs", "both"])
def test_large_ragged_batches_from_lists_in_other_orders(dgn, oracle, shuffled):
    """Waves of the build walk several times 64 operators and go from graph to graph in any lane: graphs of 0 to 230 operators, the last
    one a multiple of 64 with wide rows, whose rows come from lists of which one or both are in no order."""
    rng = np.random.default_rng(len(shuffled))
    g = recorded(rng, 5400, 230, 20, 3, 5, 4, empty_every=50)
    wide = recorded(rng, 1, 128, 40, 30, 9, 4)
    cat = lambda a, b, off: np.concatenate([a, b + off]).astype(np.int32)  # noqa: E731
    edges = [cat(g.in_op, wide.in_op, g.num_ops), cat(g.in_tensor, wide.in_tensor, g.num_tensors),
             cat(g.out_op, wide.out_op, g.num_ops), cat(g.out_tensor, wide.out_tensor, g.num_tensors)]
    for first, which in ((0, "inputs"), (2, "outputs")):
        if shuffled in (which, "both"):
            p = rng.permutation(edges[first].size)
            edges[first], edges[first + 1] = edges[first][p], edges[first + 1][p]
    P, T = g.num_ops + wide.num_ops, g.num_tensors + wide.num_tensors
    assert P > 8192 * 64 and P % 64 != 0
    h = gg.Graph(P, T, *edges, 5401, np.append(g.graph_op_offsets, P), np.append(g.graph_tensor_offsets, T), "ragged")
    dg = dgn.DeviceGraph.from_coo(h)
    adj = oracle.build_adjacency(P, T, h.in_op, h.in_tensor, h.out_op, h.out_tensor)
    for name, v in dg.csr().items():
        assert np.array_equal(v.cpu().numpy(), getattr(adj, name)), name
    # (an operator's tensors keep the order of the list: in no order they are not numbered as the sweep needs them)
    check(dgn, oracle, h, [draw_targets(rng, h, 3, 2)], swept=shuffled in ("", "inputs"))
