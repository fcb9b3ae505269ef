"""The work that a user of the library has it do, as cases that can be timed: graphs are recorded and built,
pruned for target sets, pruned backwards, and the result is read out.

Graphs are of the five families of ``graphgen`` (same recipes and distributions), generated here on the GPU so
that a 50-million-operator graph costs a fraction of a second.  Everything the path computes is whole numbers, so
results are compared exactly.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1707_08265_amd as d

NUM_INPUTS = 16           # graph inputs of every family but the layered CNN shape, whose first layer is its width
WINDOW = 64               # layered and RNN: how many of the latest tensors an input is drawn from
ZIPF_S, ZIPF_CAP = 2.1, 64


def listed():
    return [
        # One recorded step of a small model, pruned for what one call fetches: latency of a single call.
        {"name": "prune_layered_2k", "do": "prune", "graph": "layered", "ops": 2000, "sets": 1, "per_set": 4},
        # A CNN training graph, 64 choices of fetches at once: hundreds of dependent layers, medium width.
        {"name": "prune_cnn_200k", "do": "prune", "graph": "cnn", "layers": 500, "width": 400, "sets": 64, "per_set": 8},
        # An unrolled RNN of 10 000 steps, pruned for its loss and a few intermediate tensors.
        {"name": "prune_rnn_10m", "do": "prune", "graph": "rnn", "steps": 10000, "width": 1000, "sets": 1, "per_set": 33},
        # The largest single graph, power-law fan-in, 64 target sets, into buffers kept from call to call.
        {"name": "prune_powerlaw_50m", "do": "prune", "graph": "powerlaw", "ops": 50_000_000, "sets": 64, "per_set": 16},
        # More sets than one mask holds (three words, the last one ragged), on one long thin recorded graph.
        {"name": "words_layered_20k", "do": "words", "graph": "layered", "ops": 20000, "sets": 150, "per_set": 4},
        # Thousands of recorded graphs in one packed batch, 64 sets each.
        {"name": "batch_4096x20000", "do": "prune", "graph": "batch", "graphs": 4096, "ops": 20000, "ragged": False,
         "sets": 64, "per_set": 4},
        # A small packed batch of graphs of different sizes: far fewer graphs than compute units.
        {"name": "batch_96x3001_ragged", "do": "prune", "graph": "batch", "graphs": 96, "ops": 3001, "ragged": True,
         "sets": 8, "per_set": 4},
        # A graph recorded operator by operator is built into its adjacency.
        {"name": "build_ordered_50m", "do": "build", "graph": "powerlaw", "ops": 50_000_000, "order": "recorded"},
        # The same from edge lists in no order (recorded by several threads, or read from a file).
        {"name": "build_shuffled_12m", "do": "build", "graph": "powerlaw", "ops": 12_345_679, "order": "shuffled"},
        # 64 (objective, derivative target) pairs on the largest graph.
        {"name": "backward_powerlaw_50m", "do": "backward", "graph": "powerlaw", "ops": 50_000_000, "pairs": 64},
        # What follows a prune when a function is made from it: in-place names, tensors to ignore, one list per set.
        {"name": "finish_powerlaw_50m", "do": "finish", "graph": "powerlaw", "ops": 50_000_000, "sets": 64, "per_set": 16},
        # A graph that has just been recorded: built, pruned once, dropped (nothing is known from an earlier call).
        {"name": "session_cnn_200k", "do": "session", "graph": "cnn", "layers": 500, "width": 400, "sets": 64, "per_set": 8},
    ]


def _ok(rc, where):
    if rc != d.DGN_OK:
        raise d.DgnError(rc, where)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, family):
    if family == "layered":
        return {"graph": family, "ops": _log(rng, 500, 20_000)}
    if family == "cnn":
        return {"graph": family, "layers": _log(rng, 20, 1000), "width": _log(rng, 40, 800)}
    if family == "rnn":
        return {"graph": family, "steps": _log(rng, 50, 10_000), "width": _log(rng, 100, 1000)}
    if family == "batch":
        return {"graph": family, "graphs": _log(rng, 2, 4096), "ops": _log(rng, 200, 20_000), "ragged": rng.random() < 0.5}
    return {"graph": "powerlaw", "ops": _log(rng, 10_000, 50_000_000)}


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    do = rng.choice(["prune", "prune", "prune", "prune", "words", "build", "build", "backward", "finish", "session"])
    if do == "prune":
        c = _draw_graph(rng, rng.choice(["layered", "cnn", "rnn", "powerlaw", "batch"]))
        return {"do": do, **c, "sets": rng.choice([1, 64, rng.randint(2, 63)]), "per_set": rng.randint(1, 16)}
    if do == "words":
        c = _draw_graph(rng, rng.choice(["layered", "cnn", "powerlaw"]))
        if c["graph"] == "powerlaw":
            c["ops"] = min(c["ops"], _log(rng, 10_000, 4_000_000))
        return {"do": do, **c, "sets": rng.randint(65, 192), "per_set": rng.randint(1, 16)}
    if do == "build":
        c = _draw_graph(rng, rng.choice(["cnn", "rnn", "powerlaw", "batch"]))
        order = rng.choice(["recorded", "shuffled", "csr"])
        if order == "shuffled" and c["graph"] == "batch":
            order = "recorded"
        return {"do": do, **c, "order": order}
    if do == "backward":
        return {"do": do, **_draw_graph(rng, rng.choice(["layered", "cnn", "rnn", "powerlaw"])), "pairs": rng.randint(1, 64)}
    if do == "finish":
        return {"do": do, **_draw_graph(rng, rng.choice(["cnn", "rnn", "powerlaw"])),
                "sets": rng.choice([1, 64, rng.randint(2, 63)]), "per_set": rng.randint(1, 16)}
    c = _draw_graph(rng, rng.choice(["layered", "cnn"]))
    return {"do": do, **c, "sets": rng.choice([1, 64, rng.randint(2, 63)]), "per_set": rng.randint(1, 16)}


# ------------------------------------------------------------------------------------------------
# graphs on the GPU
# ------------------------------------------------------------------------------------------------
class Coo:
    """Edge lists on the device, as ``dgn_graph_build`` takes them, and what the target draws need to know."""

    def __init__(self, num_ops, num_tensors, in_op, in_tensor, out_op, out_tensor, op_off=None, t_off=None, tail_lo=0):
        self.num_ops, self.num_tensors = num_ops, num_tensors
        self.in_op, self.in_tensor, self.out_op, self.out_tensor = in_op, in_tensor, out_op, out_tensor
        self.op_off, self.t_off = op_off, t_off            # host int64, packed batches only
        self.num_graphs = 1 if op_off is None else len(op_off) - 1
        self.tail_lo = tail_lo                             # targets are drawn from [tail_lo, num_tensors)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _below(gen, n, count=None):
    """Uniform integers below n (a number, with `count` of them, or one for every element of a tensor)."""
    if isinstance(n, torch.Tensor):
        r = torch.rand(n.shape, generator=gen, device="cuda", dtype=torch.float64)
        return torch.minimum((r * n).long(), n - 1)
    return torch.randint(0, n, (count,), generator=gen, device="cuda")


def _counts(gen, base, n):
    """n counts in an order that `gen` gives; how often each occurs is fixed, so that every seed has graphs of one size.
    base: turns n uniform numbers into counts."""
    u = torch.rand(n, generator=_gen(12345), device="cuda", dtype=torch.float64)
    return base(u)[torch.randperm(n, generator=gen, device="cuda")]


def _up_to(most):
    return lambda u: 1 + (u * most).long().clamp(max=most - 1)


def _starts(counts, first=0):
    """Exclusive prefix sum of `counts`, starting at `first`."""
    return counts.cumsum(0) - counts + first


def _rows(counts):
    """Row index of every element of a ragged layout, and its slot in the row."""
    total = int(counts.sum())
    row = torch.repeat_interleave(torch.arange(counts.numel(), device="cuda"), counts, output_size=total)
    return row, torch.arange(total, device="cuda") - _starts(counts)[row]


def _window(gen, pool_first, produced, newest):
    """An input drawn from the graph's inputs (from `pool_first` on) and its last `WINDOW` tensors before `newest`."""
    r = _below(gen, NUM_INPUTS + produced.clamp(max=WINDOW))
    return torch.where(r < NUM_INPUTS, pool_first + r, newest - (r - NUM_INPUTS))


def _graph_sizes(case, seed):
    """Operators of every graph of a packed batch (host): all alike, or 0.3 to 1.7 times `ops`, in any order."""
    g, ops = case["graphs"], case["ops"]
    if not case["ragged"]:
        return np.full(g, ops, dtype=np.int64)
    sizes = np.maximum(1, (ops * (0.3 + 1.4 * (np.arange(g) + 0.5) / g)).astype(np.int64))
    return np.random.RandomState(seed % (1 << 32)).permutation(sizes)


def _record(case, seed):
    """The graph as a recorder leaves it: operator by operator."""
    gen, family = _gen(seed), case["graph"]
    op_off = t_off = None
    tail = 0.10
    if family == "cnn":
        layers, width = case["layers"], case["width"]
        P = layers * width
        n_out, fan = _counts(gen, _up_to(2), P), _counts(gen, _up_to(3), P)
        first = _starts(n_out, width)                      # `width` graph inputs stand for layer -1
        T = int(first[-1] + n_out[-1])
        starts = torch.cat([first.new_zeros(1), first[::width], first.new_tensor([T])])
        in_op, _ = _rows(fan)
        skip = torch.rand(in_op.numel(), generator=gen, device="cuda") < 0.2
        back = torch.where(skip, 2 + _below(gen, 31, in_op.numel()), 1)
        src = (in_op // width - back).clamp(min=-1) + 1
        in_t = starts[src] + _below(gen, starts[src + 1] - starts[src])
        tail_lo = int(starts[max(0, layers - 50) + 1])
    elif family == "rnn":
        width = case["width"]
        P = case["steps"] * width
        ops = torch.arange(P, device="cuda")
        n_out, fan = torch.ones_like(ops), _counts(gen, _up_to(3), P)
        rec = torch.cat([ops.new_zeros(width), _counts(gen, lambda u: (u < 0.1).long(), P - width)])
        first = ops + NUM_INPUTS
        T = P + NUM_INPUTS
        in_op, slot = _rows(fan + rec)
        own = first[in_op]
        in_t = torch.where(slot >= fan[in_op], own - width, _window(gen, 0, in_op % width, own - 1))
        tail_lo = NUM_INPUTS
    elif family == "powerlaw":
        P = case["ops"]
        cdf = torch.arange(1, ZIPF_CAP + 1, device="cuda", dtype=torch.float64).pow(-ZIPF_S).cumsum(0)
        n_out = _counts(gen, _up_to(3), P)
        fan = _counts(gen, lambda u: 1 + torch.searchsorted(cdf / cdf[-1], u, right=True).clamp(max=ZIPF_CAP - 1), P)
        first = _starts(n_out, NUM_INPUTS)
        T = int(first[-1] + n_out[-1])
        in_op, _ = _rows(fan)
        in_t = _below(gen, first[in_op])
        tail = 0.05
        tail_lo = T - max(1, int(T * tail))
    else:                                                  # layered, or a packed batch of such graphs
        sizes = _graph_sizes(case, seed) if family == "batch" else np.array([case["ops"]], dtype=np.int64)
        op_off = np.concatenate([[0], np.cumsum(sizes)])
        P = int(op_off[-1])
        of, _ = _rows(torch.from_numpy(sizes).cuda())      # graph of every operator
        n_out, fan = _counts(gen, _up_to(2), P), _counts(gen, _up_to(3), P)
        first = _starts(n_out) + NUM_INPUTS * (of + 1)
        T = int(first[-1] + n_out[-1])
        base = first[torch.from_numpy(op_off[:-1]).cuda()] - NUM_INPUTS      # first tensor of every graph
        in_op, _ = _rows(fan)
        lo, own = base[of[in_op]], first[in_op]
        in_t = _window(gen, lo, own - lo - NUM_INPUTS, own - 1)
        t_off = np.concatenate([base.cpu().numpy(), [T]])
        tail_lo = T - max(1, int(T * tail))
        if family == "layered":
            op_off = t_off = None
    out_op, slot = _rows(n_out)
    out_t = first[out_op] + slot
    i32 = lambda x: x.to(torch.int32).contiguous()  # noqa: E731
    return Coo(P, T, i32(in_op), i32(in_t), i32(out_op), i32(out_t), op_off, t_off, tail_lo), gen


def _targets(case, coo, gen):
    """`sets` target sets (per graph of a batch) of 1..per_set tensors, or exactly per_set for a single set."""
    sets, per = case["sets"], case["per_set"]
    if coo.num_graphs > 1:
        t_off = torch.from_numpy(coo.t_off).cuda()
        span = ((t_off[1:] - t_off[:-1]) // 10).clamp(min=1)
        n = torch.full((coo.num_graphs * sets,), per, device="cuda")
        g = torch.arange(coo.num_graphs * sets, device="cuda").div(sets, rounding_mode="floor").repeat_interleave(per)
        idx = t_off[1:][g] - 1 - _below(gen, span[g])
    else:
        n = 1 + _below(gen, per, sets) if sets > 1 else torch.full((1,), per, device="cuda")
        idx = coo.tail_lo + _below(gen, coo.num_tensors - coo.tail_lo, int(n.sum()))
        if case["graph"] == "rnn":
            idx[0] = coo.num_tensors - 1                   # the loss
    ptr = torch.cat([n.new_zeros(1), n.cumsum(0)])
    return ptr.to(torch.int32), idx.to(torch.int32)


def _desc(coo):
    return d.make_coo_desc(coo.num_ops, coo.num_tensors, coo.in_op, coo.in_tensor, coo.out_op, coo.out_tensor,
                           coo.num_graphs, coo.op_off, coo.t_off)


def _memory(sizes):
    rc, graph_bytes, scratch_bytes = sizes
    _ok(rc, "workspace")
    return (torch.empty(graph_bytes, dtype=torch.uint8, device="cuda"),
            torch.empty(scratch_bytes, dtype=torch.uint8, device="cuda"))


def _built(desc, mem, scratch, keep=()):
    build = d.dgn_graph_from_csr if keep else d.dgn_graph_build
    rc, handle = build(desc, mem, mem.numel(), scratch, scratch.numel())
    _ok(rc, "build")
    rc, sizes = d.dgn_graph_get_sizes(handle)
    _ok(rc, "sizes")
    return d.DeviceGraph(handle, mem, keep, sizes)


def _build(coo):
    desc = _desc(coo)
    mem, scratch = _memory(d.dgn_graph_build_workspace(desc))
    return _built(desc, mem, scratch)


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------
def _outputs(buf):
    return {"tensor_mask": buf.tensor_mask, "op_mask": buf.op_mask, "op_flag": buf.op_flag, "kept_ops": buf.kept_ops,
            "kept_masks": buf.kept_masks, "kept_count": buf.kept_count, "per_query_count": buf.per_query_count}


def _arrays(P, T, words=()):
    """Output arrays as a caller of the C interface owns them (one row per word of 64 sets)."""
    new = lambda n, t: torch.zeros(*words, n, dtype=t, device="cuda")  # noqa: E731
    return {"tensor_mask": new(T, torch.int64), "op_mask": new(P, torch.int64), "op_flag": new(P, torch.uint8),
            "kept_ops": new(P, torch.int32), "kept_masks": new(P, torch.int64), "kept_count": new(1, torch.int64),
            "per_query_count": new(64, torch.int64)}


def _clean(buf):
    """The lists are written up to their count; the rest of the arrays is given a value once, so that they can be compared whole."""
    buf.kept_ops.zero_()
    buf.kept_masks.zero_()
    return buf


def prepare(case, seed):
    coo, gen = _record(case, seed)
    do = case["do"]
    s = {"do": do}
    if do == "build":
        s["coo"], s["keep"] = coo, ()
        if case["order"] == "shuffled":
            for a, b in (("in_op", "in_tensor"), ("out_op", "out_tensor")):
                p = torch.randperm(getattr(coo, a).numel(), generator=gen, device="cuda")
                setattr(coo, a, getattr(coo, a)[p])
                setattr(coo, b, getattr(coo, b)[p])
        if case["order"] == "csr":
            ptr = lambda key: torch.searchsorted(key, torch.arange(coo.num_ops + 1, device="cuda", dtype=torch.int32)).to(torch.int32)  # noqa: E731
            s["keep"] = (ptr(coo.in_op), coo.in_tensor, ptr(coo.out_op), coo.out_tensor)
            s["desc"] = d.make_csr_desc(coo.num_ops, coo.num_tensors, *s["keep"], coo.num_graphs, coo.op_off, coo.t_off)
            s["mem"], s["scratch"] = _memory(d.dgn_graph_from_csr_workspace(s["desc"]))
        else:
            s["desc"] = _desc(coo)
            s["mem"], s["scratch"] = _memory(d.dgn_graph_build_workspace(s["desc"]))
        return s
    if do == "session":
        s["coo"] = coo
        s["targets"] = _targets(case, coo, gen)
        s["sets"], s["out"] = case["sets"], _arrays(coo.num_ops, coo.num_tensors)
        return s
    graph = s["graph"] = _build(coo)
    if do == "backward":
        sources = case["width"] if case["graph"] == "cnn" else NUM_INPUTS
        span = max(1, int(graph.num_tensors * 0.05))
        s["pairs"] = (_below(gen, sources, case["pairs"]).to(torch.int32),
                      (graph.num_tensors - span + _below(gen, span, case["pairs"])).to(torch.int32))
        s["buf"] = _clean(d.BackwardPruneBuffers(graph, case["pairs"]))
        return s
    s["targets"] = _targets(case, coo, gen)
    if do == "words":
        rc, bytes_ = d.dgn_prune_workspace(graph.handle, 64)
        _ok(rc, "workspace")
        s["sets"], s["scratch"] = case["sets"], torch.empty(bytes_, dtype=torch.uint8, device="cuda")
        s["out"] = _arrays(graph.num_ops, graph.num_tensors, ((case["sets"] + 63) // 64,))
        return s
    s["buf"] = _clean(d.PruneBuffers(graph, case["sets"]))
    if do == "finish":
        _ok(s["buf"].prune(*s["targets"]), "prune")
        s["inplace"], s["read"] = d.InplaceBuffers(graph), d.ReadoutBuffers(s["buf"])
        # room for the lists of every seed's result
        most = min(graph.num_ops, 2 * int(_expected(case)[3]) + 1000)
        s["read"].set_ops = torch.zeros(most * case["sets"], dtype=torch.int32, device="cuda")
    return s


def _pruned(graph, s, scratch, entry):
    (ptr, idx), o = s["targets"], s["out"]
    return entry(graph.handle, s["sets"], idx.numel(), ptr, idx, o["tensor_mask"], o["op_mask"], o["op_flag"],
                 o["kept_ops"], o["kept_masks"], o["kept_count"], o["per_query_count"], scratch, scratch.numel())


def run(s):
    do = s["do"]
    if do == "prune":
        _ok(s["buf"].prune(*s["targets"]), "prune")
        return _outputs(s["buf"])
    if do == "words":
        _ok(_pruned(s["graph"], s, s["scratch"], d.dgn_prune_words), "prune_words")
        return s["out"]
    if do == "build":
        graph = _built(s["desc"], s["mem"], s["scratch"], s["keep"])
        out = graph.csr()
        graph.close()
        return out
    if do == "backward":
        _ok(s["buf"].backward_prune(*s["pairs"]), "backward_prune")
        return _outputs(s["buf"])
    if do == "finish":
        b, i, r = s["buf"], s["inplace"], s["read"]
        _ok(i.run(b.op_mask, kept_ops=b.kept_ops, kept_count=b.kept_count), "inplace")
        _ok(r.ignore(), "ignore")
        _ok(r.per_set_lists(), "per_set_lists")
        return {"rename": i.rename, "renamed_count": i.renamed_count, "ignore_mask": r.ignore_mask,
                "ignore_count": r.ignore_count, "set_rowptr": r.set_rowptr, "set_ops": r.set_ops}
    graph = _build(s["coo"])                               # session: built, pruned once, the count read, dropped
    rc, bytes_ = d.dgn_prune_workspace(graph.handle, s["sets"])
    _ok(rc, "workspace")
    _ok(_pruned(graph, s, torch.empty(bytes_, dtype=torch.uint8, device="cuda"), d.dgn_prune), "prune")
    kept = int(s["out"]["kept_count"][0])
    graph.close()
    return {**s["out"], "kept": kept}


def _expected(case):
    """Expected (operators, tensors, input edges, kept operators, targets)."""
    family = case["graph"]
    if family == "powerlaw":
        w = [k ** -ZIPF_S for k in range(1, ZIPF_CAP + 1)]
        P, outs, fan = case["ops"], 2.0, sum(k * x for k, x in enumerate(w, 1)) / sum(w)
    elif family == "cnn":
        P, outs, fan = case["layers"] * case["width"], 1.5, 2.0
    elif family == "rnn":
        P, outs, fan = case["steps"] * case["width"], 1.0, 2.1
    else:
        P, outs, fan = case["ops"] * case.get("graphs", 1), 1.5, 2.0
    targets = case.get("sets", case.get("pairs", 1)) * (case.get("per_set", 1) + 1) / 2 * case.get("graphs", 1)
    # Power law: an operator at id y is needed with the density (targets * fan / P) * (P / y)^fan, so about all below
    # the id where that reaches one are kept.  RNN: about the neighbourhood of a target.  Else nearly everything.
    kept = P
    if family == "powerlaw":
        kept = min(P, 1.15 * P * (fan * targets / P) ** (1 / fan))
    elif family == "rnn":
        kept = min(P, targets * case["width"])
    return P, P * outs, P * fan, kept, targets


def work(case):
    """Bytes that the path cannot do without (there is no floating-point work).

    A prune: the rows of the kept operators (two row bounds and the ids) and the targets read, and of the outputs --
    masks of tensors and operators, a flag byte, the list with its masks -- what is not zero, once; `words` and
    `session` write into arrays that hold nothing yet, so all of those.  A build: the edge lists read, the three
    adjacency lists with their row pointers written.  Reading out: the kept list and its rows read, the rename
    dictionary and the ignore mask written in full, and the lists."""
    P, T, E, kept, targets = _expected(case)
    outs, fan = T / P, E / P
    rows = kept * (8 + 4 * fan + 4 * outs)
    result = kept * (8 * outs + 8 + 1 + 12)
    do = case["do"]
    build = 2 * 4 * (E + T) + 4 * (E + 2 * T) + 4 * (2 * P + T)
    if do == "build":
        b = build - (4 * (E + T + P) + 4 * (E + T) if case["order"] == "csr" else 0)
    elif do == "words":
        b = rows * (case["sets"] + 63) // 64 + ((case["sets"] + 63) // 64) * (8 * T + 9 * P + 12 * kept)
    elif do == "session":
        b = build + rows + 8 * T + 9 * P + 12 * kept
    elif do == "finish":
        b = rows + kept * (12 + 8 * outs) + 4 * T + 8 * T + 4 * kept * case["sets"] / 2
    else:
        b = rows + result + 4 * targets
    return {"bytes": float(b), "flops": 0.0}


def tolerance(case):
    return "exact"
