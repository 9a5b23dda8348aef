"""The workloads this repository's speed is judged by.

A case is one mini-batch of dataflow graphs and the way a program runs it:

* ``call: False``: the prepared path (``edb.Forward``): the program keeps the
  graph, schedule, plan and packed weights of a mini-batch and runs its
  forward pass (training epochs over kept mini-batches, fixed-shape serving).
* ``call: True``: the whole path for a new input graph in one call
  (``edb.ForwardCall``): ingest, schedule, plan, descriptors and execution.

``config`` names the model family of ``workloads.make_config`` (the shapes of
the graphs are its distributions), ``instances`` the graphs in the mini-batch,
``in_dim`` and ``hidden`` the sizes, ``dtype`` the storage of W, x and h.
A pass returns both state arenas whole: every node's h and c.
"""
from __future__ import annotations

import dataclasses
import functools

import numpy as np
import torch

from paper_2302_03851_amd import _lib as L
from paper_2302_03851_amd import edb
from paper_2302_03851_amd import workloads as WL

# weight scale of each family's synthetic configuration, and its dimensions
SCALE = {1: 0.1, 2: 0.08, 3: 0.1, 4: 0.08, 5: 0.05, 6: 0.08, 7: 0.08, 9: 0.1}
DIMS = {1: (64, 64), 2: (256, 256), 3: (100, 200), 4: (128, 256), 5: (512, 512), 6: (256, 256), 7: (256, 256),
        8: (64, 64), 9: (100, 200)}
# arena rows a program provides per graph: room for the family's largest graph
ROWS = {1: 20, 2: 100, 3: 120, 4: 288, 5: 600, 6: 100, 7: 100, 8: 100 * 65, 9: 180}
GATES = {WL.LSTM_CHAIN: 4, WL.NARY_LEAF: 3, WL.NARY_INTERNAL: 5, WL.GRID: 5, WL.CS_LEAF: 3, WL.CS_INTERNAL: 3,
         WL.LAT_CHAR: 4, WL.LAT_WORD: 3, WL.GRU_LEAF: 2, WL.GRU_INTERNAL: 3, WL.LINEAR: 1, WL.MV_MAT: 1,
         WL.MV_VEC: 1, WL.LGRU_EDGE: 3, WL.POOL_MEAN: 1}


def _case(name, config, instances, in_dim=None, hidden=None, dtype=None, call=False):
    e, h = DIMS[config]
    return {"name": name, "config": config, "instances": instances, "in_dim": in_dim or e, "hidden": hidden or h,
            "dtype": dtype or ("bf16" if config == 5 else "f32"), "call": call}


def listed():
    return [
        # a tagger over a handful of short sentences: the smallest call
        _case("chain_8", 1, 8),
        # a bucket of sentences in one encoder layer, 16-bit weights
        _case("chain_128_bf16", 1, 128, 256, 256, "bf16"),
        # sentiment / parsing trees: the reference workload, kept mini-batch
        _case("tree_64", 2, 64),
        # the same for a mini-batch not seen before, graph work included
        _case("tree_64_call", 2, 64, call=True),
        # a large training mini-batch of trees
        _case("tree_1024", 2, 1024),
        # named-entity lattices (characters and lexicon words)
        _case("lattice_32", 3, 32),
        # image-like grids: wide anti-diagonal wavefronts
        _case("grid_32", 4, 32),
        # large child-sum trees, 16-bit weights: the largest contraction
        _case("childsum_256_bf16", 5, 256),
        # a serving-sized mini-batch of new child-sum trees
        _case("childsum_16_bf16_call", 5, 16, call=True),
        # trees of gated recurrent units
        _case("treegru_64", 7, 64),
        # matrix-vector trees: many small products
        _case("mvrnn_64", 8, 64),
        # lattices of gated recurrent units, pooled per position
        _case("lattice_gru_32", 9, 32),
    ]


def draw(rng):
    """A case of the same ranges: any family, from one graph to a large
    mini-batch, sizes from 32 to 512 (320 where a batch has 5 gates over
    several operands) with ragged ones among them, either way to run it."""
    config = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 9])
    top = {1: 256, 2: 256, 3: 64, 4: 32, 5: 128, 6: 256, 7: 256, 8: 96, 9: 64}[config]
    instances = max(1, round(top ** rng.random()))
    dtype = "bf16" if config == 5 or (config < 8 and rng.random() < 0.3) else "f32"
    step = 8 if dtype == "bf16" else 4
    e, h = DIMS[config]
    if config != 8 and rng.random() < 0.7:   # an MV-RNN's d is part of its graph
        limit = 512 if config in (1, 5) else 320
        h = max(32, round(32 * (limit / 32) ** rng.random() / step) * step)
        e = max(32, round(32 * (limit / 32) ** rng.random() / step) * step)
    e = -(-e // step) * step   # rows of whole 16 bytes
    return {"config": config, "instances": instances, "in_dim": e, "hidden": h, "dtype": dtype,
            "call": rng.random() < 0.25}


def _workload(case, seed):
    """The mini-batch: make_config's graphs, with weights and inputs redrawn
    from its distributions where the sizes or the type are other ones."""
    k, E, H = case["config"], case["in_dim"], case["hidden"]
    w = WL.make_config(k, seed=seed, instances=case["instances"])
    if (E, H) == (w.in_dim, w.hidden) and case["dtype"] == w.dtype:
        return w
    rng = np.random.default_rng(seed)
    cast = WL.round_bf16 if case["dtype"] == "bf16" else (lambda m: m)
    weights = []
    for t, kind in enumerate(w.kinds):
        d = {}
        for name, shape in WL.weight_shapes(kind, E, H, w.n_children[t] or 2):
            if name.startswith("b"):
                d[name] = np.zeros(shape, dtype=np.float32)
            elif kind == WL.POOL_MEAN:
                d[name] = np.eye(H, dtype=np.float32)
            else:
                d[name] = cast(rng.uniform(-SCALE[k], SCALE[k], size=shape).astype(np.float32))
        weights.append(d)
    x = cast(rng.standard_normal(size=(w.x.shape[0], E), dtype=np.float32))
    return dataclasses.replace(w, in_dim=E, hidden=H, dtype=case["dtype"], weights=weights, x=x)


def _rows(case):
    return 64 + case["instances"] * ROWS[case["config"]]


def prepare(case, seed):
    w = _workload(case, seed)
    f = edb.Forward(w, device="cuda")
    # one pair of arenas for mini-batches of varying size
    if f.plan.n_slots > _rows(case):
        raise ValueError("the mini-batch does not fit the arenas")
    f.arena_h = torch.zeros((_rows(case), w.hidden), dtype=f.tdt, device="cuda")
    f.arena_c = torch.zeros((_rows(case), w.hidden), dtype=torch.float32, device="cuda")
    if not case["call"]:
        return {"f": f}
    table = edb.LATTICE_TABLE if case["config"] == 3 else None
    call = edb.ForwardCall(w.op_type, w.child_ptr, w.child_idx, w.x_row, w.n_types, edb.operand_shapes(w), f.cells,
                           table=table)
    return {"f": f, "call": call, "w": [b.data_ptr() for b in f.weights]}


def run(state):
    f = state["f"]
    if "call" in state:
        state["call"].call(state["w"], f.x.data_ptr(), f.arena_h.data_ptr(), f.arena_c.data_ptr(),
                           f.arena_h.shape[0], f.stream.cuda_stream)
    else:
        f.run()
    return {"h": f.arena_h, "c": f.arena_c}


@functools.lru_cache(maxsize=64)
def _work(key):
    case = dict(key)
    w = WL.make_config(case["config"], seed=0, instances=case["instances"])
    E, H, V = case["in_dim"], case["hidden"], w.n_nodes
    esz = 2 if case["dtype"] == "bf16" else 4
    flops = 0
    n_children = np.diff(w.child_ptr)
    present = np.add.reduceat(np.append(w.child_idx, -1) >= 0, np.minimum(w.child_ptr[:-1], w.child_idx.size))
    present = np.where(n_children > 0, present, 0)
    for t, kind in enumerate(w.kinds):
        rows = w.op_type == t
        n, kids = int(rows.sum()), int(present[rows].sum())
        g = GATES[kind]
        if kind in (WL.LINEAR, WL.POOL_MEAN):
            continue                                         # identity maps
        if kind == WL.CS_INTERNAL:
            flops += n * 2 * H * 3 * H + kids * 2 * H * H
        elif kind == WL.LAT_CHAR:
            first = w.child_idx[w.child_ptr[:-1][rows]]
            prev, words = int((first >= 0).sum()), kids - int((first >= 0).sum())
            flops += (n * E + prev * H) * 2 * g * H + words * 2 * H * H
        elif kind == WL.MV_VEC:
            flops += n * (4 * H * H + 4 * H * H)
        elif kind == WL.GRU_INTERNAL:
            flops += kids * 2 * H * (g + 1) * H
        else:
            flops += ((n * E if WL.KIND_SHAPE[kind][2] else 0) + kids * H) * 2 * g * H
    n_x = int((w.x_row >= 0).sum())
    weights = sum(int(np.prod(s)) for t, kind in enumerate(w.kinds)
                  for _, s in WL.weight_shapes(kind, E, H, w.n_children[t] or 2))
    return {"bytes": weights * esz + n_x * E * esz + V * H * (esz + 4), "flops": float(flops)}


def work(case):
    return dict(_work(tuple(sorted((k, v) for k, v in case.items() if k != "name"))))


def tolerance(case):
    # four times the largest error against exact() over the listed cases and six
    # drawn ones: 1.7e-3 (h rounded to bf16 at every node) and 5.7e-7 (the grids)
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 0.05}
    return {"rel": 2.4e-6, "max": 4e-5}


def exact(case, seed):
    """The states in 64 bits, node by node of one depth at a time, laid out in
    the arenas' rows (the plan's slots; row 0 and pad rows are zero)."""
    w = _workload(case, seed)
    dev = torch.device("cuda")
    H, V = w.hidden, w.n_nodes
    deg = np.diff(w.child_ptr)
    parent = np.repeat(np.arange(V), deg)
    here = w.child_idx >= 0
    depth = np.zeros(V, dtype=np.int64)
    while True:
        new = depth.copy()
        np.maximum.at(new, parent[here], depth[w.child_idx[here]] + 1)
        if np.array_equal(new, depth):
            break
        depth = new
    x = torch.from_numpy(np.ascontiguousarray(w.x)).to(dev).double()
    Wt = [{n: torch.from_numpy(m).to(dev).double() for n, m in d.items()} for d in w.weights]
    h = torch.zeros((V + 1, H), dtype=torch.float64, device=dev)   # row V (index -1): the absent child
    c = torch.zeros_like(h)
    sg, th = torch.sigmoid, torch.tanh
    order = np.lexsort((w.op_type, depth))
    cut = np.flatnonzero(np.diff(depth[order]) | np.diff(w.op_type[order])) + 1
    for rows in np.split(order, cut):
        kind, p = w.kinds[w.op_type[rows[0]]], Wt[w.op_type[rows[0]]]
        fixed = {WL.NARY_INTERNAL: 2}.get(kind, WL.KIND_SHAPE[kind][0])
        at = torch.from_numpy(rows).to(dev)
        kid = [torch.from_numpy(w.child_idx[w.child_ptr[rows] + i].astype(np.int64)).to(dev) for i in range(fixed)]
        xr = x[torch.from_numpy(w.x_row[rows].astype(np.int64)).to(dev)] if WL.KIND_SHAPE[kind][2] else None
        a = torch.cat(([xr] if xr is not None else []) + [h[i] for i in kid], dim=1) if xr is not None or kid else None
        ragged = [], []                                            # row in `rows`, child
        if WL.KIND_SHAPE[kind][1] and kind != WL.MV_VEC:
            for i, v in enumerate(rows):
                ch = w.child_idx[w.child_ptr[v] + fixed:w.child_ptr[v + 1]]
                ch = ch[ch >= 0]
                ragged[0].extend([i] * len(ch))
                ragged[1].extend(ch.tolist())
        owner, child = (torch.tensor(r, dtype=torch.int64, device=dev) for r in ragged)
        if kind in (WL.LSTM_CHAIN, WL.NARY_LEAF, WL.CS_LEAF, WL.NARY_INTERNAL, WL.GRID, WL.LAT_WORD):
            z = (a @ p["W"] + p["b"]).split(H, dim=1)
            if kind == WL.LSTM_CHAIN:
                nc = sg(z[1]) * c[kid[0]] + sg(z[0]) * th(z[2])
                nh = sg(z[3]) * th(nc)
            elif kind in (WL.NARY_LEAF, WL.CS_LEAF):
                nc = sg(z[0]) * th(z[2])
                nh = sg(z[1]) * th(nc)
            elif kind == WL.LAT_WORD:
                nc = sg(z[1]) * c[kid[0]] + sg(z[0]) * th(z[2])
                nh = torch.zeros_like(nc)
            else:
                nc = sg(z[0]) * th(z[4]) + sg(z[1]) * c[kid[0]] + sg(z[2]) * c[kid[1]]
                nh = sg(z[3]) * th(nc)
        elif kind == WL.CS_INTERNAL:
            hs = torch.zeros((len(rows), H), dtype=torch.float64, device=dev).index_add_(0, owner, h[child])
            z = (hs @ p["U_iou"] + p["b_iou"]).split(H, dim=1)
            fc = sg(h[child] @ p["U_f"] + p["b_f"]) * c[child]
            nc = (sg(z[0]) * th(z[2])).index_add_(0, owner, fc)
            nh = sg(z[1]) * th(nc)
        elif kind == WL.LAT_CHAR:
            z = (a @ p["W"] + p["b"]).split(H, dim=1)
            e = torch.exp(sg(xr[owner] @ p["W_lx"] + c[child] @ p["W_lc"] + p["b_l"]))
            e0 = torch.exp(sg(z[0]))
            num = (e0 * th(z[3])).index_add_(0, owner, e * c[child])
            den = e0.clone().index_add_(0, owner, e)
            worded = torch.zeros(len(rows), dtype=torch.bool, device=dev)
            worded[owner] = True
            nc = torch.where(worded[:, None], num / den, sg(z[1]) * c[kid[0]] + sg(z[0]) * th(z[3]))
            nh = sg(z[2]) * th(nc)
        elif kind == WL.GRU_LEAF:
            z = (a @ p["W"] + p["b"]).split(H, dim=1)
            nc = nh = (1 - sg(z[0])) * th(z[1])
        elif kind == WL.GRU_INTERNAL:
            h0, h1 = h[kid[0]], h[kid[1]]
            z = (a @ p["W"][:, :3 * H] + p["b"][:3 * H]).split(H, dim=1)
            n0 = h0 @ p["W"][:H, 3 * H:4 * H] + p["b"][3 * H:4 * H]
            n1 = h1 @ p["W"][H:, 4 * H:] + p["b"][4 * H:]
            nc = nh = sg(z[0]) * (h0 + h1) / 2 + (1 - sg(z[0])) * th(sg(z[1]) * n0 + sg(z[2]) * n1)
        elif kind == WL.LINEAR:
            nc = nh = a @ p["W"] + p["b"]
        elif kind == WL.MV_MAT:
            nc = nh = a @ p["W_M"] + p["b"]
        elif kind == WL.MV_VEC:
            cols = np.stack([w.child_idx[w.child_ptr[v] + 2:w.child_ptr[v + 1]] for v in rows]).astype(np.int64)
            A, B = (h[torch.from_numpy(np.ascontiguousarray(q)).to(dev)] for q in (cols[:, :H], cols[:, H:]))
            ba = (h[kid[0]][:, :, None] * B).sum(1)
            ab = (h[kid[1]][:, :, None] * A).sum(1)
            nc = nh = th(torch.cat([ba, ab], dim=1) @ p["W"] + p["b"])
        elif kind == WL.LGRU_EDGE:
            hs, E = h[kid[0]], w.in_dim
            z = (a @ p["W"][:, :2 * H] + p["b"][:2 * H]).split(H, dim=1)
            nx = xr @ p["W"][:E, 2 * H:3 * H] + p["b"][2 * H:3 * H]
            nhs = hs @ p["W"][E:, 3 * H:] + p["b"][3 * H:]
            nc = nh = (1 - sg(z[0])) * th(nx + sg(z[1]) * nhs) + sg(z[0]) * hs
        else:  # POOL_MEAN
            s = torch.zeros((len(rows), H), dtype=torch.float64, device=dev).index_add_(0, owner, h[child])
            n = torch.zeros(len(rows), dtype=torch.float64, device=dev).index_add_(
                0, owner, torch.ones(len(child), dtype=torch.float64, device=dev))
            nc = nh = (s / n.clamp(min=1)[:, None]) @ p["W"] + p["b"]
        h[at], c[at] = nh, nc
    f = edb.Forward(w, flags=L.DRYRUN)   # the schedule and plan alone: where each node's row lies
    slot = torch.from_numpy(f.plan.slot.astype(np.int64)).to(dev)
    out = {}
    for name, s in (("h", h), ("c", c)):
        out[name] = torch.zeros((_rows(case), H), dtype=torch.float64, device=dev)
        out[name][slot] = s[:V]
    return out
