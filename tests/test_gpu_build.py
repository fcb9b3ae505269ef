"""GPU parity of the builder's pass over the edge lists: lists in operator order (finished by it alone), gaps between rows at
the lengths where they are left to another pass, tensors with several producers, and lists in other orders; the
adjacency against the oracle's, and records and producer words through a prune that reads them."""
import numpy as np
import pytest

import graphgen as gg
from helpers import targets_from_sets
from test_gpu_parity import assert_same, oracle_prune

pytestmark = pytest.mark.gpu
ROWS = ("in_rowptr", "in_idx", "out_rowptr", "out_idx", "prod_rowptr", "prod_idx")


@pytest.fixture(scope="module")
def dgn():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_1707_08265_amd as d
    return d


def listed(rng, writers, first_gap, gap, several):
    """`writers` operators that write one tensor each, `gap` tensors without producer and as many operators without outputs
    between two of them here and there, first_gap such tensors and operators before the first; several: some tensors are
    written by the next operators too."""
    hole = rng.random(writers) < (0.1 if gap else 0)
    step = 1 + hole * gap
    op = first_gap + np.cumsum(step) - step[0]
    t = first_gap + 1 + np.cumsum(step) - step[0]
    P, T = int(op[-1]) + 1 + gap, int(t[-1]) + 1 + gap
    out_op, out_t = op, t
    if several:
        more = rng.integers(0, 3, writers) * (rng.random(writers) < 0.3)
        which = np.repeat(np.arange(writers), 1 + more)
        out_t = t[which]
        out_op = op[np.minimum(which + np.arange(which.size) - np.searchsorted(which, which), writers - 1)]
        order = np.argsort(out_op, kind="stable")
        out_op, out_t = out_op[order], out_t[order]
    fan = rng.integers(0, 4, writers)
    in_op = np.repeat(op, fan)
    in_t = (rng.random(in_op.size) * np.repeat(t, fan)).astype(np.int64)
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    return gg.Graph(P, T, i32(in_op), i32(in_t), i32(out_op), i32(out_t), name="listed")


def check(dgn, oracle, g, rng, what):
    import torch
    sets = [[int(x) for x in rng.integers(0, g.num_tensors, 3)] for _ in range(7)]
    tg = targets_from_sets(sets, 7)
    adj, ref = oracle_prune(oracle, g, tg)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    for borrowed in (False, True):
        if borrowed:
            desc = dgn.make_csr_desc(g.num_ops, g.num_tensors, *(keep := [up(getattr(adj, n)) for n in ROWS[:4]]))
            rc, mem, scratch = dgn.dgn_graph_from_csr_workspace(desc)
            mem, scratch = (torch.full((n,), 255, dtype=torch.uint8, device="cuda") for n in (mem, scratch))
            rc, handle = dgn.dgn_graph_from_csr(desc, mem, mem.numel(), scratch, scratch.numel())
            assert rc == 0, dgn.dgn_strerror(rc)
            dg = dgn.DeviceGraph(handle, mem, keep, dgn.dgn_graph_get_sizes(handle)[1])
        else:
            dg = dgn.DeviceGraph.from_coo(g)
        csr = {n: v.cpu().numpy() for n, v in dg.csr().items()}
        for name in ROWS:
            assert np.array_equal(csr[name], getattr(adj, name)), f"{what}, borrowed {borrowed}: {name}"
        buf = dgn.PruneBuffers(dg, 7)
        rc = buf.prune(up(tg.tgt_rowptr), up(tg.tgt_idx), options=dgn.dgn_options(traversal=1))
        assert rc == 0
        assert_same(buf.to_host(), ref, f"{what}, borrowed {borrowed}")


@pytest.mark.parametrize("several", [False, True])
@pytest.mark.parametrize("shape", [(1, 0, 0), (3, 1, 0), (4, 3, 0), (255, 5, 1), (1023, 16, 2), (1024, 0, 63), (1025, 7, 64),
                                   (3000, 8190, 65), (5000, 8191, 3), (4096, 8192, 0), (140_000, 16, 0), (90_000, 3, 70)])
def test_lists_in_order(dgn, oracle, shape, several):
    rng = np.random.default_rng(sum(shape) + several)
    check(dgn, oracle, listed(rng, *shape, several), rng, f"{shape}")


@pytest.mark.parametrize("several", [None, "first", "last", "all"])
@pytest.mark.parametrize("writers,at", [(9, 4), (63, 62), (64, 1), (65, 64), (1025, 1), (4096, 4093), (5003, 1024), (140_000, 69_999), (140_001, 3)])
def test_outputs_in_two_runs(dgn, oracle, writers, at, several):
    """One hole in the numbering: producer words that the pass over the outputs has left out for what it took for one run, up to
    the last tensor, are filled in; with tensors of several producers before or behind the hole, also more outputs than tensors."""
    rng = np.random.default_rng(writers + at)
    t = 5 + np.arange(writers) + 2 * (np.arange(writers) >= at)
    op, more = np.arange(writers), np.zeros(writers, dtype=np.int64)
    if several:
        more[{"first": 0, "last": writers - 1, "all": slice(None)}[several]] = 1
    out_t, fan = np.repeat(t, 1 + more), rng.integers(0, 3, writers)
    out_op = np.minimum(np.repeat(op, 1 + more) + np.concatenate([np.arange(n) for n in (1 + more)]), writers - 1)
    in_op = np.repeat(op, fan)
    in_t = (rng.random(in_op.size) * np.repeat(t, fan)).astype(np.int64)
    order = np.argsort(out_op, kind="stable")
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    g = gg.Graph(writers, int(t[-1]) + 1, i32(in_op), i32(in_t), i32(out_op[order]), i32(out_t[order]), name="two runs")
    check(dgn, oracle, g, rng, f"{writers} {at} {several}")


@pytest.mark.parametrize("numbering", ["run", "in rows", "hole"])
@pytest.mark.parametrize("ops,fan,at", [(1, 0, 1), (3, 0, 0), (1023, 1, 1), (1024, 0, 2), (1025, 2, 3), (5000, 2, 0), (140_000, 1, 1)])
def test_borrowed_rows_of_any_alignment(dgn, oracle, ops, fan, at, numbering):
    """Borrowed arrays that begin `at` entries past a 16-byte boundary, with and without inputs, sizes around a workgroup's entries: outputs that
    are one run of tensors (finished without a pass over them as a list), that are one but for the order inside rows, and that have a hole."""
    import torch
    rng = np.random.default_rng(ops + at)
    n_out = rng.integers(0, 3, ops)
    n_out[-1] = 2
    t = 4 + np.arange(n_out.sum())
    out_op, in_op = np.repeat(np.arange(ops), n_out), np.repeat(np.arange(ops), fan)
    own = 4 + np.concatenate([[0], np.cumsum(n_out)])[:-1]   # first output, so that inputs are others' outputs or the four graph inputs
    in_t = own[in_op] - 1 - (rng.random(in_op.size) * np.minimum(own[in_op], 300)).astype(np.int64)
    if numbering == "in rows":
        t[-2:] = t[-2:][::-1]
    if numbering == "hole":
        in_t += in_t >= t[len(t) // 2]
        t[len(t) // 2:] += 1
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    g = gg.Graph(ops, int(t.max()) + 1, i32(in_op), i32(in_t), i32(out_op), i32(t), name="borrowed")
    tg = targets_from_sets([[int(x) for x in rng.integers(0, g.num_tensors, 3)] for _ in range(5)], 5)
    adj, ref = oracle_prune(oracle, g, tg)
    assert fan == 0 or ops < 1000 or np.count_nonzero(ref.op_mask) > 3 * 15, "the prune stops at the targets' own producers"
    keep = []
    for name in ROWS[:4]:
        a = torch.zeros(getattr(adj, name).size + at, dtype=torch.int32, device="cuda")[at:]
        keep.append(a.copy_(torch.from_numpy(np.ascontiguousarray(getattr(adj, name)))))
    dg = dgn.DeviceGraph.from_csr(g.num_ops, g.num_tensors, *keep)
    csr = {n: v.cpu().numpy() for n, v in dg.csr().items()}
    for name in ROWS:
        assert np.array_equal(csr[name], getattr(adj, name)), name
    buf = dgn.PruneBuffers(dg, 5)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    assert buf.prune(up(tg.tgt_rowptr), up(tg.tgt_idx), options=dgn.dgn_options(traversal=1)) == 0
    assert_same(buf.to_host(), ref, numbering)


@pytest.mark.parametrize("nnz", [8192 * 1024, 8192 * 1024 + 1, 8192 * 1024 + 77])
@pytest.mark.parametrize("order", ["recorded", "outputs", "inputs", "last"])
def test_long_lists_are_looked_at_before(dgn, oracle, nnz, order):
    """Lists up to and beyond the length from which a few places are looked at first: in order, one of them in no order, and a
    single pair at the end, which that look does not see."""
    import torch
    P = (nnz + 1) // 2
    per = np.full(P, 2)
    per[0] += nnz - 2 * P
    op = np.repeat(np.arange(P), per).astype(np.int32)
    t = np.arange(nnz, dtype=np.int32) + 3
    in_t = (np.arange(nnz, dtype=np.int64) * 7919 % (op.astype(np.int64) * 2 + 3)).astype(np.int32)
    rng = np.random.default_rng(nnz)
    pi, po = np.arange(nnz), np.arange(nnz)
    if order == "inputs":
        pi = rng.permutation(nnz)
    if order == "outputs":
        po = rng.permutation(nnz)
    if order == "last":
        po[[-1, -3]] = po[[-3, -1]]
    g = gg.Graph(P, nnz + 3, op[pi], in_t[pi], op[po], t[po], name="long")
    adj = oracle.build_adjacency(g.num_ops, g.num_tensors, g.in_op, g.in_tensor, g.out_op, g.out_tensor)
    csr = {n: v.cpu().numpy() for n, v in dgn.DeviceGraph.from_coo(g).csr().items()}
    for name in ROWS:
        assert np.array_equal(csr[name], getattr(adj, name)), f"{order}: {name}"
    g.in_op[nnz // 3] = P                                    # an id out of range, wherever the lists are left early
    from paper_1707_08265_amd import DgnError
    with pytest.raises(DgnError):
        dgn.DeviceGraph.from_coo(g)
    torch.cuda.synchronize()


@pytest.mark.parametrize("most", [1, 3, 4, 5, 9, 63, 64, 65, 200])
def test_shuffled_outputs_of_operators_with_many(dgn, oracle, most):
    """Rows inside and beyond what a thread holds, up to the longest that is ordered without a sort and above."""
    rng = np.random.default_rng(most)
    n_out = rng.integers(0, most + 1, 400)
    n_out[7] = most
    P, T = n_out.size, int(n_out.sum()) + 3
    out_op, out_t = np.repeat(np.arange(P), n_out), 3 + np.arange(n_out.sum())
    in_op = np.arange(P)
    in_t = (rng.random(P) * (3 + np.cumsum(n_out) - n_out)).astype(np.int64)
    p = rng.permutation(out_op.size)
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    check(dgn, oracle, gg.Graph(P, T, i32(in_op), i32(in_t), i32(out_op[p]), i32(out_t[p]), name="rows"), rng, f"{most}")


@pytest.mark.parametrize("several", [False, True])
@pytest.mark.parametrize("order", ["outputs", "inputs", "all", "halves", "tensors", "one"])
def test_lists_in_other_orders(dgn, oracle, order, several):
    """Outputs that are back in order by tensor once they are sorted by operator, and outputs that are not."""
    rng = np.random.default_rng(17 + several)
    for shape in ((700, 5, 2), (150_000, 16, 0)):
        g = listed(rng, *shape, several)
        ni, no = g.nnz_in, g.nnz_out
        pi, po = np.arange(ni), np.arange(no)
        if order in ("inputs", "all"):
            pi = rng.permutation(ni)
        if order in ("outputs", "all"):
            po = rng.permutation(no)
        if order == "halves":                    # two threads' recordings, one behind the other
            pi, po = np.concatenate([pi[1::2], pi[::2]]), np.concatenate([po[1::2], po[::2]])
        if order == "one":                       # a single pair out of order
            po[no // 2], po[no // 2 + 1] = po[no // 2 + 1], po[no // 2]
        if order == "tensors":                   # operators in order, tensors not
            g.out_tensor[:] = rng.permutation(g.out_tensor)
        h = gg.Graph(g.num_ops, g.num_tensors, g.in_op[pi], g.in_tensor[pi], g.out_op[po], g.out_tensor[po], name=order)
        check(dgn, oracle, h, rng, f"{order} {shape}")


def _shuffled(rng, n_out, fan, inputs=5, numbering="created"):
    """An operator per entry: how many tensors it writes and reads; both lists in no order."""
    P, E = n_out.size, int(n_out.sum())
    first = inputs + np.cumsum(n_out) - n_out
    T = inputs + E
    in_op, out_op, out_t = np.repeat(np.arange(P), fan), np.repeat(np.arange(P), n_out), inputs + np.arange(E)
    in_t = (rng.random(in_op.size) * first[in_op]).astype(np.int64)
    if numbering == "gaps":                        # every other tensor, ascending: not one run
        T, in_t, out_t = 2 * T, 2 * in_t, 2 * out_t
    elif numbering == "mixed":                     # tensors of neighbouring operators change places
        far = np.arange(E)
        far[: E // 2 * 2] = far[: E // 2 * 2].reshape(-1, 2)[:, ::-1].ravel()
        out_t = out_t[far]
    elif numbering == "twice":                     # one tensor written by two operators, one by none
        out_t[E // 2] = out_t[E // 2 - 1]
    elif numbering == "more":                      # more outputs than tensors
        T, in_t, out_t = T // 2 + 1, in_t // 2, out_t // 2
    pi, po = rng.permutation(in_op.size), rng.permutation(E)
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    return gg.Graph(P, int(T), i32(in_op[pi]), i32(in_t[pi]), i32(out_op[po]), i32(out_t[po]), name="shuffled")


@pytest.mark.parametrize("numbering", ["created", "gaps", "mixed", "twice", "more"])
@pytest.mark.parametrize("ops, outs, fan", [(3, 2, 3), (64, 1, 1), (511, 3, 3), (512, 2, 2), (1025, 2, 2), (16384, 1, 0), (16385, 1, 1),
                                            (70_001, 2, 5), (150_001, 1, 3), (300_000, 1, 2), (300_000, 0.03, 0.05)])
def test_lists_sorted_by_buckets(dgn, oracle, ops, outs, fan, numbering):
    """One bucket, one tile and one more, ragged last buckets, sparse rows, one pass and two into buckets."""
    rng = np.random.default_rng(ops)
    count = lambda mean: rng.integers(0, 2 * mean + 1, ops) if mean >= 1 else (rng.random(ops) < mean).astype(np.int64)  # noqa: E731
    n_out = count(outs)
    n_out[:3] = 1, 2, 1
    check(dgn, oracle, _shuffled(rng, n_out, count(fan), numbering=numbering), rng, f"{ops} {outs} {fan} {numbering}")


@pytest.mark.parametrize("order", ["one", "halves", "two", "three", "runs"])
@pytest.mark.parametrize("ops, outs, fan", [(4097, 2, 2), (12_293, 2, 3), (100_001, 1, 2), (300, 90, 150)])
def test_lists_nearly_in_order(dgn, oracle, ops, outs, fan, order):
    """Neighbouring keys have the same digits: in all lanes of a wave, of two recordings or three taken in turn, or of one now and
    then; sorted by buckets and as a whole (few operators with many tensors)."""
    rng = np.random.default_rng(ops)
    n_out = rng.integers(0, 2 * outs + 1, ops)
    n_out[:3] = 1, 2, 1
    g = _shuffled(rng, n_out, rng.integers(0, 2 * fan + 1, ops))

    def placed(op, t):
        by = np.argsort(op, kind="stable")
        op, t, n = op[by], t[by], op.size
        p = np.arange(n)
        if order == "one":
            p[[n // 2, n // 3]] = p[[n // 3, n // 2]]
        elif order == "halves":
            p = np.concatenate([p[1::2], p[::2]])
        elif order in ("two", "three"):
            k = 2 if order == "two" else 3
            p = np.concatenate([p[:n // k * k].reshape(k, -1).T.ravel(), p[n // k * k:]])
        else:                                          # stretches of 1 to 900 edges change places
            cut = np.split(p, np.cumsum(rng.integers(1, 901, n // 450)).clip(0, n))
            p = np.concatenate([cut[i] for i in rng.permutation(len(cut))])
        return op[p], t[p]
    h = gg.Graph(g.num_ops, g.num_tensors, *placed(g.in_op, g.in_tensor), *placed(g.out_op, g.out_tensor), name=order)
    check(dgn, oracle, h, rng, f"{ops} {order}")


@pytest.mark.parametrize("which", ["inputs", "outputs"])
@pytest.mark.parametrize("most, rows", [(2048, 1), (2049, 1), (4097, 2), (14_000, 1), (30_000, 1), (30_000, 3), (131_072, 1), (17_000, 70)])
def test_rows_of_several_tiles_and_many_large_buckets(dgn, oracle, most, rows, which):
    """Operators with so many inputs or outputs that their bucket is done in tiles by one workgroup or by several."""
    rng = np.random.default_rng(most)
    n_out, fan = rng.integers(0, 3, 40_000), rng.integers(0, 4, 40_000)
    (fan if which == "inputs" else n_out)[39_999 - 571 * np.arange(rows)] = most
    check(dgn, oracle, _shuffled(rng, n_out, fan), rng, f"{which} {most}")


@pytest.mark.parametrize("which", ["inputs", "outputs"])
@pytest.mark.parametrize("ops, most, rows", [(40_000, 17_000, 257), (40_000, 34_817, 60), (300_000, 2_100_000, 1), (300_000, 500_000, 3)])
def test_more_large_buckets_than_threads_and_very_large_ones(dgn, oracle, ops, most, rows, which):
    """Their tiles are counted in groups, from nine tiles (three groups) to a thousand."""
    rng = np.random.default_rng(most)
    n_out, fan = rng.integers(0, 3, ops), rng.integers(0, 4, ops)
    (fan if which == "inputs" else n_out)[ops - 1 - ops // rows * np.arange(rows)] = most
    check(dgn, oracle, _shuffled(rng, n_out, fan), rng, f"{which} {most}")


@pytest.mark.parametrize("ops, outs, fan", [(3, 2, 3), (900, 1, 2), (200, 90, 90), (70_001, 2, 5), (300_000, 1, 2), (300_000, 0.03, 0.05)])
def test_ids_out_of_range_in_lists_in_no_order(dgn, ops, outs, fan):
    """One id out of range anywhere in either list is reported and nothing is built (the first pass sees all of lists this short)."""
    import torch
    rng = np.random.default_rng(ops)
    count = lambda mean: rng.integers(0, 2 * mean + 1, ops) if mean >= 1 else (rng.random(ops) < mean).astype(np.int64)  # noqa: E731
    n_out, fans = count(outs), count(fan)
    n_out[:3], fans[:3] = 2, 2
    good = _shuffled(rng, n_out, fans)
    for name, limit in (("in_op", good.num_ops), ("in_tensor", good.num_tensors), ("out_op", good.num_ops), ("out_tensor", good.num_tensors)):
        for bad in (-1, limit, -(1 << 31), (1 << 31) - 1):
            lists = {n: getattr(good, n).copy() for n in ("in_op", "in_tensor", "out_op", "out_tensor")}
            lists[name][rng.integers(lists[name].size)] = bad
            up = {n: torch.from_numpy(v).cuda() for n, v in lists.items()}
            desc = dgn.make_coo_desc(good.num_ops, good.num_tensors, *up.values(), 1, None, None)
            rc, mem, scratch = dgn.dgn_graph_build_workspace(desc)
            mem, scratch = (torch.full((n,), 255, dtype=torch.uint8, device="cuda") for n in (mem, scratch))
            print(ops, name, bad, flush=True)
            rc, handle = dgn.dgn_graph_build(desc, mem, mem.numel(), scratch, scratch.numel())
            assert rc == dgn.DGN_ERR_ID_OUT_OF_RANGE, (name, bad, rc)


@pytest.mark.parametrize("which", ["inputs", "outputs"])
def test_many_tensors_out_of_range_beside_rows_of_several_tiles(dgn, which):
    """Workgroups that rank rows report such tensors while others begin with theirs, some of them with buckets of more than one tile:
    the call says so and writes nothing beside its memory.  The list is longer than the 8 388 608 edges that the first pass has looked at
    when its last wave has taken its first step (a wave that has met a decrease takes no other)."""
    import torch
    rng = np.random.default_rng(5)
    ops = 4_400_000
    count = np.full(ops, 2)
    count[999_999::1_000_000] = 2049, 10_000, 100_000, 17_000
    one, many = np.arange(ops), np.repeat(np.arange(ops), count)
    if which == "inputs":
        in_op, out_op = rng.permutation(many), one
        in_t = (rng.random(in_op.size) * (5 + in_op)).astype(np.int64)
        out_t = 5 + one
    else:
        order = rng.permutation(many.size)
        in_op, in_t, out_op, out_t = one, np.zeros(ops, np.int64), many[order], 5 + order
    num_tensors = 5 + out_op.size
    bad_list = in_t if which == "inputs" else out_t
    at = (1 << 23) + rng.choice(bad_list.size - (1 << 23), 3000, replace=False)
    was = bad_list[at].copy()
    margin = 1 << 16
    for bad in (True, False):
        bad_list[at] = num_tensors + rng.integers(0, 1 << 28, at.size) if bad else was
        up = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda() for a in (in_op, in_t, out_op, out_t)]
        desc = dgn.make_coo_desc(ops, num_tensors, *up, 1, None, None)
        rc, *need = dgn.dgn_graph_build_workspace(desc)
        memory = [torch.full((n + margin,), 0xab, dtype=torch.uint8, device="cuda") for n in need]
        print(which, bad, flush=True)
        rc, handle = dgn.dgn_graph_build(desc, memory[0], need[0], memory[1], need[1])
        assert rc == (dgn.DGN_ERR_ID_OUT_OF_RANGE if bad else dgn.DGN_OK)
        for m, n in zip(memory, need):
            assert bool((m[n:] == 0xab).all())
        if handle:
            dgn.dgn_graph_destroy(handle)


_LONG = {}


def _long_lists(ops, each):
    """Lists in operator order in which every operator reads and writes `each` tensors: more than 8 388 608 edges, which is what the first
    pass has looked at when its last wave has taken its first step (a wave that has met a decrease takes no other)."""
    if (ops, each) not in _LONG:
        _LONG.clear()
        op = np.repeat(np.arange(ops, dtype=np.int32), each)
        t = np.arange(op.size, dtype=np.int32)
        assert op.size > (1 << 23) + 1000
        _LONG[ops, each] = op, (np.random.default_rng(ops).random(op.size) * (5 + op.astype(np.int64) * each)).astype(np.int32), 5 + t
    return _LONG[ops, each]


@pytest.mark.parametrize("inputs, outputs", [("shuffled", "ordered"), ("shuffled", "mixed"), ("shuffled", "gaps"), ("shuffled", "shuffled"),
                                             ("ordered", "shuffled")])
@pytest.mark.parametrize("ops, each", [(20_000, 460), (4_300_000, 2)])
def test_ids_out_of_range_late_in_long_lists(dgn, ops, each, inputs, outputs):
    """Ids that only the sorts come to see, of lists that are sorted as a whole and by buckets: reported, and nothing is made of rows
    that were not written.  What the memory held stays inside the lists if it is taken for rows by tensor (a row with an entry, a
    row before it, ...); "mixed" is the list of which the first pass writes no such row, so that no word says "no producer" then."""
    import torch
    rng = np.random.default_rng(ops)
    op, in_t, out_t = _long_lists(ops, each)
    num_tensors = op.size + 5
    pi, po = (rng.permutation(op.size) if order == "shuffled" else slice(None) for order in (inputs, outputs))
    if outputs == "mixed":
        out_t = 5 + rng.permutation(op.size).astype(np.int32)
    elif outputs == "gaps":                                    # 70 tensors without producer every thousand
        out_t = out_t + out_t // 1000 * 70
        num_tensors = int(out_t[-1]) + 1
    good = {"in_op": op[pi], "in_tensor": in_t[pi], "out_op": op[po], "out_tensor": out_t[po]}
    up = {n: torch.from_numpy(np.ascontiguousarray(v)).cuda() for n, v in good.items()}
    desc = dgn.make_coo_desc(ops, num_tensors, *up.values(), 1, None, None)
    rc, mem, scratch = dgn.dgn_graph_build_workspace(desc)
    mem, scratch = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (mem, scratch))
    words = mem[:mem.numel() // 8 * 8].view(torch.int32)
    for name in good:
        if (inputs if name.startswith("in") else outputs) != "shuffled":
            continue
        for bad in (ops if name.endswith("op") else num_tensors, 1 << 30):
            at = op.size - int(rng.integers(1, 1000))
            print(ops, inputs, outputs, name, bad, at, flush=True)
            was = int(up[name][at])
            up[name][at] = bad
            words[0::2], words[1::2] = 0, 1
            scratch.fill_(0)
            rc, handle = dgn.dgn_graph_build(desc, mem, mem.numel(), scratch, scratch.numel())
            assert rc == dgn.DGN_ERR_ID_OUT_OF_RANGE, (name, bad, rc)
            assert outputs != "mixed" or not bool((words < 0).any())
            up[name][at] = was
    rc, handle = dgn.dgn_graph_build(desc, mem, mem.numel(), scratch, scratch.numel())
    assert rc == dgn.DGN_OK
    dgn.dgn_graph_destroy(handle)


@pytest.mark.parametrize("validate", [0, 1])
@pytest.mark.parametrize("ops", [1, 700, 150_000])
def test_faults_of_a_borrowed_csr_are_reported_wherever_they_are(dgn, oracle, ops, validate):
    """The arrays are checked by the device and what follows is enqueued behind that: no kernel trusts rows that are none."""
    import torch
    rng = np.random.default_rng(ops)
    g = listed(rng, ops, 0, 0, False)
    adj = oracle.build_adjacency(g.num_ops, g.num_tensors, g.in_op, g.in_tensor, g.out_op, g.out_tensor)
    good = {n: np.ascontiguousarray(getattr(adj, n)) for n in ROWS[:4]}
    cases = [("out_rowptr", 0, 1, "csr"), ("out_rowptr", g.num_ops, -7, "csr"), ("in_rowptr", g.num_ops, (1 << 31) - 1, "csr"),
             ("out_rowptr", g.num_ops // 2, (1 << 31) - 1, "csr"), ("in_rowptr", g.num_ops // 2, -1, "csr"),
             ("out_idx", g.nnz_out // 2, -1, "id"), ("out_idx", g.nnz_out - 1, g.num_tensors, "id"), (None, 0, 0, None)]
    if g.nnz_in:
        cases += [("in_idx", g.nnz_in - 1, g.num_tensors, "id"), ("in_idx", 0, -(1 << 31), "id")]
    for name, at, value, what in cases:
        arrays = {n: v.copy() for n, v in good.items()}
        if name:
            arrays[name][at] = value
        keep = [torch.from_numpy(v).cuda() for v in arrays.values()]
        desc = dgn.make_csr_desc(g.num_ops, g.num_tensors, *keep)
        rc, mem, scratch = dgn.dgn_graph_from_csr_workspace(desc)
        mem, scratch = (torch.full((n,), 255, dtype=torch.uint8, device="cuda") for n in (mem, scratch))
        print(ops, name, at, value, flush=True)
        rc, handle = dgn.dgn_graph_from_csr(desc, mem, mem.numel(), scratch, scratch.numel(), dgn.dgn_options(validate=validate))
        want = {"csr": dgn.DGN_ERR_BAD_CSR, "id": dgn.DGN_ERR_ID_OUT_OF_RANGE, None: dgn.DGN_OK}[what]
        assert rc == want, (name, at, value, rc)
        if handle:
            dgn.dgn_graph_destroy(handle)


@pytest.mark.parametrize("graphs", [63, 64, 65, 200])
@pytest.mark.parametrize("relabelled", [False, True])
def test_batches_around_the_number_that_have_no_records(dgn, oracle, graphs, relabelled):
    """From 64 graphs on a batch has a word per operator in the place of records: levels, in-place pass (from op_mask and from the list) and ignore mask
    go by it, also where an operator's outputs are not consecutive."""
    import torch
    g, tg = gg.batch_layered(graphs, 150, 77 + graphs, num_sets=7, per_set=3)
    if relabelled:                                           # the tensors of every graph in another order
        rng = np.random.default_rng(graphs)
        off = g.graph_tensor_offsets
        new = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(off[:-1], off[1:])]).astype(np.int32)
        g = gg.Graph(g.num_ops, g.num_tensors, g.in_op, new[g.in_tensor], g.out_op, new[g.out_tensor], g.num_graphs, g.graph_op_offsets, off, "relabelled")
        tg = gg.Targets(tg.num_sets, tg.tgt_rowptr, new[tg.tgt_idx])
    adj, ref = oracle_prune(oracle, g, tg)
    dg = dgn.DeviceGraph.from_coo(g)
    buf = dgn.PruneBuffers(dg, 7)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    assert buf.prune(up(tg.tgt_rowptr), up(tg.tgt_idx), options=dgn.dgn_options(traversal=1)) == 0
    assert_same(buf.to_host(), ref, "levels")
    few = dgn.PruneBuffers(dg, 7)                            # more targets than the queues hold: every operator is looked at until nothing changes
    assert few.prune(up(tg.tgt_rowptr), up(tg.tgt_idx), options=dgn.dgn_options(traversal=1, max_queue_entries=16)) == 0
    assert_same(few.to_host(), ref, "queues that overflow")
    ip, ro = dgn.InplaceBuffers(dg), dgn.ReadoutBuffers(buf)
    want = oracle.inplace(adj, ref.op_mask, (1 << 64) - 1)
    for how in ({}, {"kept_ops": buf.kept_ops, "kept_count": buf.kept_count}):
        assert ip.run(buf.op_mask, **how) == 0
        assert np.array_equal(ip.rename.cpu().numpy(), want), f"in-place {list(how)}"
    assert ro.ignore() == 0
    assert np.array_equal(ro.ignore_mask.cpu().numpy().view(np.uint64), oracle.ignore_mask(adj, ref.op_mask, ref.tensor_mask))


@pytest.mark.parametrize("largest", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("relabelled", [False, True])
def test_batches_with_a_graph_around_the_largest_that_is_swept(dgn, oracle, largest, relabelled):
    """A batch of 64 graphs goes level by level, with operator records, if one of them is larger than that, and is swept, without, if none is; both
    ways the prune that nobody asks for levels, the in-place pass and the ignore mask agree with the oracle."""
    import torch
    rng = np.random.default_rng(largest + relabelled)
    sizes = rng.integers(1, 60, 64)
    sizes[rng.integers(0, 64)] = largest
    P, off = int(sizes.sum()), np.concatenate([[0], np.cumsum(sizes)])
    of = np.repeat(np.arange(64), sizes)
    n_out, fan = rng.integers(1, 3, P), rng.integers(1, 4, P)
    first = np.concatenate([[0], np.cumsum(n_out)])[:-1] + 3 * (of + 1)       # three inputs per graph in front of its outputs
    T = int(n_out.sum()) + 3 * 64
    t_off = np.concatenate([first[off[:-1]] - 3, [T]]).astype(np.int64)
    in_op, out_op = np.repeat(np.arange(P), fan), np.repeat(np.arange(P), n_out)
    back = np.minimum(first[in_op] - t_off[of[in_op]], 300)                   # outputs of the last few operators, or the inputs
    in_t = first[in_op] - 1 - (rng.random(in_op.size) * back).astype(np.int64)
    out_t = first[out_op] + np.concatenate([np.arange(n) for n in n_out])
    new = np.arange(T)
    if relabelled:
        new = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(t_off[:-1], t_off[1:])])
    i32 = lambda a: np.ascontiguousarray(a, dtype=np.int32)  # noqa: E731
    g = gg.Graph(P, T, i32(in_op), i32(new[in_t]), i32(out_op), i32(new[out_t]), 64, off.astype(np.int64), t_off, "one large")
    sets = [[int(new[hi - 1 - rng.integers(0, min(hi - lo, 20))])] for lo, hi in zip(t_off[:-1], t_off[1:]) for _ in range(3)]
    tg = gg.Targets(3, i32(np.arange(len(sets) + 1)), i32(np.concatenate(sets)))
    adj, ref = oracle_prune(oracle, g, tg)
    dg = dgn.DeviceGraph.from_coo(g)
    buf, st = dgn.PruneBuffers(dg, 3), dgn.dgn_stats()
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    for call in range(2):
        assert buf.prune(up(tg.tgt_rowptr), up(tg.tgt_idx), stats=st) == 0
        assert_same(buf.to_host(), ref, f"call {call}")
        assert (st.levels > 1) == (largest > 1 << 18), st.levels
    ip, ro = dgn.InplaceBuffers(dg), dgn.ReadoutBuffers(buf)
    want = oracle.inplace(adj, ref.op_mask, (1 << 64) - 1)
    for how in ({}, {"kept_ops": buf.kept_ops, "kept_count": buf.kept_count}):
        assert ip.run(buf.op_mask, **how) == 0
        assert np.array_equal(ip.rename.cpu().numpy(), want), f"in-place {list(how)}"
    assert ro.ignore() == 0
    assert np.array_equal(ro.ignore_mask.cpu().numpy().view(np.uint64), oracle.ignore_mask(adj, ref.op_mask, ref.tensor_mask))


@pytest.mark.parametrize("shape", ["small", "large", "layers", "batch"])
@pytest.mark.parametrize("source", ["ordered", "hole", "shuffled", "borrowed", "borrowed hole"])
def test_memory_at_eight_bytes(dgn, oracle, shape, source):
    """Storage, scratch and outputs that begin eight bytes past a 16-byte boundary, which is all that the interface asks for: graphs that are swept, in
    layers, traversed, and packed batches."""
    import torch
    rng = np.random.default_rng(len(shape) + len(source))
    if shape == "batch":
        g, tg = gg.batch_layered(70, 333, 5, num_sets=7, per_set=3)
    else:
        ops = {"small": 2003, "large": 140_003, "layers": 24_000}[shape]
        o, n_out = np.arange(ops), rng.integers(1, 3, ops)
        first = 5 + np.concatenate([[0], np.cumsum(n_out)])
        op = np.repeat(o, 2)
        lo = first[np.maximum(op // 400 - 2, 0) * 400] if shape == "layers" else np.zeros(op.size)
        hi = first[op // 400 * 400] if shape == "layers" else first[op]
        in_t = np.where(hi > lo, lo + rng.random(op.size) * (hi - lo), rng.integers(0, 5, op.size)).astype(np.int32)
        g = gg.Graph(ops, int(first[-1]), op.astype(np.int32), in_t, np.repeat(o, n_out).astype(np.int32), np.arange(5, first[-1], dtype=np.int32), name=shape)
        tg = targets_from_sets([[int(x) for x in rng.integers(0, g.num_tensors, 3)] for _ in range(7)], 7)
    if "hole" in source and shape != "batch":               # a tensor that nobody writes, behind half of the outputs
        at = int(g.out_tensor[g.nnz_out // 2])
        up1 = lambda a: (a + (a >= at)).astype(np.int32)  # noqa: E731
        g = gg.Graph(g.num_ops, g.num_tensors + 1, g.in_op, up1(g.in_tensor), g.out_op, up1(g.out_tensor), name="hole")
        tg = gg.Targets(tg.num_sets, tg.tgt_rowptr, up1(tg.tgt_idx))
    adj, ref = oracle_prune(oracle, g, tg)
    if source == "shuffled":
        p, q = rng.permutation(g.nnz_in), rng.permutation(g.nnz_out)
        g = gg.Graph(g.num_ops, g.num_tensors, g.in_op[p], g.in_tensor[p], g.out_op[q], g.out_tensor[q], g.num_graphs, g.graph_op_offsets,
                     g.graph_tensor_offsets, "shuffled")
        adj = oracle.build_adjacency(g.num_ops, g.num_tensors, g.in_op, g.in_tensor, g.out_op, g.out_tensor)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    at8 = lambda n, t=torch.uint8: torch.zeros(n * t.itemsize + 8, dtype=torch.uint8, device="cuda")[8:].view(t)  # noqa: E731
    print(shape, source, flush=True)
    if "borrowed" in source:
        keep = [up(getattr(adj, n)) for n in ROWS[:4]]
        desc = dgn.make_csr_desc(g.num_ops, g.num_tensors, *keep, g.num_graphs, g.graph_op_offsets, g.graph_tensor_offsets)
        query, build = dgn.dgn_graph_from_csr_workspace, dgn.dgn_graph_from_csr
    else:
        keep, lists = (), [up(a) for a in (g.in_op, g.in_tensor, g.out_op, g.out_tensor)]
        desc = dgn.make_coo_desc(g.num_ops, g.num_tensors, *lists, g.num_graphs, g.graph_op_offsets, g.graph_tensor_offsets)
        query, build = dgn.dgn_graph_build_workspace, dgn.dgn_graph_build
    rc, *sizes = query(desc)
    mem, scratch = (at8(n) for n in sizes)
    assert mem.data_ptr() % 16 == scratch.data_ptr() % 16 == 8
    rc, handle = build(desc, mem, mem.numel(), scratch, scratch.numel())
    assert rc == 0, dgn.dgn_strerror(rc)
    dg = dgn.DeviceGraph(handle, mem, keep, dgn.dgn_graph_get_sizes(handle)[1])
    csr = {n: v.cpu().numpy() for n, v in dg.csr().items()}
    for name in ROWS:
        assert np.array_equal(csr[name], getattr(adj, name)), name
    buf = dgn.PruneBuffers(dg, tg.num_sets)
    buf.scratch = at8(buf.scratch_bytes)
    for name in ("tensor_mask", "op_mask", "op_flag", "kept_masks", "kept_count", "per_query_count"):
        setattr(buf, name, at8(getattr(buf, name).numel(), getattr(buf, name).dtype))
    for options in (None, None, dgn.dgn_options(traversal=1)):
        assert buf.prune(up(tg.tgt_rowptr), up(tg.tgt_idx), options=options) == 0
        assert_same(buf.to_host(), ref, f"levels {options is not None}")
    ip, ro = dgn.InplaceBuffers(dg), dgn.ReadoutBuffers(buf)
    ip.scratch = at8(ip.scratch_bytes)
    for how in ({}, {"kept_ops": buf.kept_ops, "kept_count": buf.kept_count}):
        assert ip.run(buf.op_mask, **how) == 0
        assert np.array_equal(ip.rename.cpu().numpy(), oracle.inplace(adj, ref.op_mask, (1 << 64) - 1)), f"in-place {list(how)}"
    assert ro.ignore() == 0
    assert np.array_equal(ro.ignore_mask.cpu().numpy().view(np.uint64), oracle.ignore_mask(adj, ref.op_mask, ref.tensor_mask))
