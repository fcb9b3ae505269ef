"""Which deferral schedule a graph gets, read from the level trace: results never depend on it, times do (the measurements
stand beside the rule in api.hip)."""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgn():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_1707_08265_amd as d
    return d


def targets(g, family, per_set, sets):
    """In the last fifth; an unrolled RNN's anywhere (its chains of operators are short)."""
    return gg.targets_range(3, sets, per_set, per_set, 16 if family == "rnn" else int(g.num_tensors * 0.8), g.num_tensors)


def thresholds(dgn, g, tg, **knobs):
    import torch
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), tg.num_sets)
    trace = np.full((512, 4), -7, np.int32)
    st = dgn.dgn_stats()
    st.level_trace, st.level_trace_cap = trace.ctypes.data, trace.shape[0]
    rc = buf.prune(torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda(),
                   options=dgn.dgn_options(traversal=1, **knobs), stats=st)
    assert rc == 0, dgn.dgn_strerror(rc)
    return trace[:int(st.levels), 2]


# (family, sizes, targets per set, sets, waits only down to an eighth of the graph): layers too few for that, a handful of
# targets in a hundred layers and many of them, enough layers, so many of them that sets and width count as well, reads from all over the graph, an RNN with few and
# many targets
@pytest.mark.parametrize("family,size,per_set,sets,soon", [
    ("cnn", (24, 700), 8, 1, False), ("cnn", (24, 700), 8, 64, False), ("cnn", (100, 300), 8, 1, False),
    ("cnn", (100, 300), 8, 64, True), ("cnn", (150, 120), 1, 64, False), ("cnn", (250, 200), 8, 1, True),
    ("cnn", (250, 200), 1, 64, True), ("cnn", (500, 200), 8, 1, True), ("cnn", (950, 100), 8, 1, False),
    ("cnn", (950, 100), 4, 4, False), ("cnn", (950, 100), 8, 9, True), ("cnn", (950, 500), 8, 1, True),
    ("powerlaw", (200_000,), 1, 64, False), ("rnn", (400, 200), 4, 64, False), ("rnn", (400, 200), 9, 64, True)])
def test_floor_of_the_thresholds(dgn, family, size, per_set, sets, soon):
    g = gg.cnn(*size, 5)[0] if family == "cnn" else gg.rnn(*size, 5) if family == "rnn" else gg.powerlaw(*size, 5)
    tg = targets(g, family, per_set, sets)
    theta = thresholds(dgn, g, tg)
    lowest = int(theta[theta > 0].min())
    floor = max(64, g.num_ops >> 10)
    assert lowest >= g.num_ops >> 3 if soon else lowest < 4 * floor, theta     # (one level takes at most 0.7 of a threshold)
    # nothing is known of a graph whose tensors are numbered in another order, and a floor of the caller's stands
    g2, t2, _ = gg.relabel_tensors(g, tg, 7)
    theta = thresholds(dgn, g2, t2)
    assert int(theta[theta > 0].min()) < 4 * floor, theta
    theta = thresholds(dgn, g, tg, defer_floor_shift=2)
    assert int(theta[theta > 0].min()) >= g.num_ops >> 2, theta


@pytest.mark.parametrize("per_set,soon", [(3, False), (8, True)])
def test_words_of_sets_count_their_own_targets(dgn, per_set, soon):
    """Two words of 64 sets on 100 layers: 192 targets each are few, whatever the call has in all; 512 are many."""
    import torch
    g = gg.cnn(100, 300, 5)[0]
    tg = targets(g, "cnn", per_set, 128)
    P, T, words = g.num_ops, g.num_tensors, 2
    graph = dgn.DeviceGraph.from_coo(g)
    rc, size = dgn.dgn_prune_workspace(graph.handle, 64)
    assert rc == 0
    new = lambda n, t: torch.zeros(words, n, dtype=t, device="cuda")  # noqa: E731
    trace = np.full((512, 4), -7, np.int32)
    st = dgn.dgn_stats()
    st.level_trace, st.level_trace_cap = trace.ctypes.data, trace.shape[0]
    rc = dgn.dgn_prune_words(graph.handle, 128, len(tg.tgt_idx), torch.from_numpy(tg.tgt_rowptr).cuda(),
                             torch.from_numpy(tg.tgt_idx).cuda(), new(T, torch.int64), new(P, torch.int64), new(P, torch.uint8),
                             new(P, torch.int32), new(P, torch.int64), new(1, torch.int64), new(64, torch.int64),
                             torch.empty(size, dtype=torch.uint8, device="cuda"), size, stats=st)
    assert rc == 0, dgn.dgn_strerror(rc)
    theta = trace[:, 2]                                                  # (the last word's levels, at least)
    lowest = int(theta[theta > 0].min())
    assert lowest >= P >> 3 if soon else lowest < P >> 6, theta


@pytest.mark.parametrize("size,per_set,sets", [((2000, 139), 4, 64), ((700, 150), 4, 64), ((60, 300), 6, 17), ((400, 200), 8, 64), ((1000, 100), 8, 64)])
def test_repeated_prunes_settle_on_one_way(dgn, oracle, size, per_set, sets):
    """Frontiers of a few hundred in a deep graph: the first prune may be done by the one workgroup, later ones start with wide
    launches, and from then on nothing changes any more (no call takes the other way, or a second batch)."""
    import torch
    g = gg.rnn(*size, 5)
    tg = gg.targets_range(3, sets, 1, per_set, 16, g.num_tensors)
    buf = dgn.PruneBuffers(dgn.DeviceGraph.from_coo(g), sets)
    ptr, idx = torch.from_numpy(tg.tgt_rowptr).cuda(), torch.from_numpy(tg.tgt_idx).cuda()
    seen = []
    for _ in range(12):
        st = dgn.dgn_stats()
        assert buf.prune(ptr, idx, stats=st) == 0
        seen.append((int(st.launches), int(st.level_launches), int(st.max_frontier)))
    if seen[0][2] <= 1024:
        assert seen[0][1] == 0, seen                        # one workgroup, no wide launch ahead of knowing
    # (the spare launches behind the layout go once it has fitted a few times)
    assert max(n for n, _, _ in seen[1:]) <= 20 and len({n for n, _, _ in seen[7:]}) == 1, seen
    adj = oracle.build_adjacency(g.num_ops, g.num_tensors, g.in_op, g.in_tensor, g.out_op, g.out_tensor)
    ref = oracle.forward_prune(adj, sets, tg.tgt_rowptr, tg.tgt_idx)
    assert np.array_equal(buf.to_host()["kept_masks"][:int(ref.kept_count[0])], ref.kept_masks[:int(ref.kept_count[0])])


@pytest.mark.parametrize("sets", [1, 64])
@pytest.mark.parametrize("extra", [0, 1, 511, 2049, 5 * 2048 + 8])
def test_count_of_kept_operators_from_their_flags(dgn, oracle, extra, sets):
    """Graphs of 4 194 304 operators and more, whose kept operators lie densely in a few tiles (chains at both ends) and thinly
    elsewhere, with last tiles of all kinds."""
    from helpers import targets_from_sets
    from test_gpu_parity import assert_same, gpu_prune, oracle_prune
    rng = np.random.default_rng(extra + sets)
    P = (1 << 22) + extra
    ops = np.arange(P)
    before = np.minimum(ops, 3000 + ops // 9)
    in_t = np.where((ops < 6000) | (ops >= P - 5000), ops - 1 + 16, (rng.random(P) * (16 + before)).astype(np.int64))
    in_t[P - 5000] = 7
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    g = gg.Graph(P, P + 16, i32(ops), i32(in_t), i32(ops), i32(ops + 16), name="flags")
    far = [int(x) for x in rng.integers(6000, P - 5000, 40)]
    tg = targets_from_sets([[P + 15 - 64 * q, 16 + far[q % 40], 16 + 5999 - q] for q in range(sets)], sets)
    _, _, out = gpu_prune(dgn, g, tg)
    _, ref = oracle_prune(oracle, g, tg)
    assert_same(out, ref, f"{extra} {sets}")
