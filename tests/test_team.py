"""Team launches: the tail of a schedule as one launch whose work-groups keep
their units' weights in registers and exchange h rows through the arena.
CPU: the planned descriptors validate.  GPU: parity with the oracle at the
edges of the kernels (widths, row remainders, absent and many children), NaN
states, teams walked alone and several in flight."""
import functools

import numpy as np
import pytest

from oracle.compare import state_rel_err
from oracle.evaluate import evaluate_workload
from paper_2302_03851_amd import _lib as L
from paper_2302_03851_amd import edb
from paper_2302_03851_amd import workloads as WL


def _graph(kinds, E, H, dtype, seed, op, ch, hx):
    return WL.make_graph(kinds, E, H, op, ch, hx, seed=seed, dtype=dtype, bias_scale=0.2)


def _chains(E, H, dtype, lengths, seed):
    op, ch = [], []
    for n in lengths:
        for t in range(n):
            op.append(0)
            ch.append([-1 if t == 0 else len(op) - 2])
    return _graph([WL.LSTM_CHAIN], E, H, dtype, seed, op, ch, [True] * len(op))


def _trees(kinds, E, H, dtype, n_trees, depth, seed):
    """Trees that grow by one leaf a level (deep schedules), with an absent
    child now and then; three kinds: internal nodes of two types in turn."""
    rng = np.random.default_rng(seed)
    op, ch, hx = [], [], []
    for t in range(n_trees):
        op.append(0), ch.append([]), hx.append(True)
        top = len(op) - 1
        for d in range(depth - t % 3):
            if rng.random() < 0.2:
                other = -1
            else:
                op.append(0), ch.append([]), hx.append(True)
                other = len(op) - 1
            pair = [top, other] if rng.random() < 0.5 else [other, top]
            op.append(1 if len(kinds) == 2 else 1 + (d + t) % 2), ch.append(pair), hx.append(False)
            top = len(op) - 1
    return _graph(kinds, E, H, dtype, seed, op, ch, hx)


def _grids(E, H, dtype, n, R, C, seed):
    op, ch = [], []
    for _ in range(n):
        base = len(op)
        for i in range(R):
            for j in range(C):
                op.append(0)
                ch.append([base + i * C + j - 1 if j else -1, base + (i - 1) * C + j if i else -1])
    return _graph([WL.GRID], E, H, dtype, seed, op, ch, [True] * len(op))


def _lattices(kinds, E, H, dtype, n, length, words, seed):
    """Characters with `words` words ending at every third of them."""
    op, ch, hx = [], [], []
    gru = kinds[0] == WL.LGRU_EDGE
    for _ in range(n):
        prev, back = -1, []
        for j in range(length):
            ends = [back[max(0, j - 1 - k % 3)] for k in range(words)] if j and j % 3 == 0 else []
            if gru:
                edges = []
                for src in [prev] + ends:
                    op.append(0), ch.append([src]), hx.append(True)
                    edges.append(len(op) - 1)
                op.append(1), ch.append(edges), hx.append(False)
            else:
                ws = []
                for src in ends:
                    op.append(1), ch.append([src]), hx.append(True)
                    ws.append(len(op) - 1)
                op.append(0), ch.append([prev] + ws), hx.append(True)
            prev = len(op) - 1
            back.append(prev)
    return _graph(kinds, E, H, dtype, seed, op, ch, hx)


def _mixed_lattices(E, H, dtype, n, length, how, seed):
    """Lattices whose links stray from characters and words in turn: `how`
    "char" gives a character the one two back as a ragged child, "word" ends a
    word in a word (its positional child), "after" follows a word with a
    character (the character's positional child)."""
    op, ch, hx = [], [], []
    for _ in range(n):
        prev, back = -1, []
        for j in range(length):
            rag = [back[j - 2]] if how == "char" and j >= 2 else []
            if how != "char" and j % 3 == 2:
                op.append(1), ch.append([back[j - 2]]), hx.append(True)
                word = len(op) - 1
                if how == "word":
                    op.append(1), ch.append([word]), hx.append(True)
                    word = len(op) - 1
                if how == "after":
                    prev = word
                else:
                    rag = [word]
            op.append(0), ch.append([prev] + rag), hx.append(True)
            prev = len(op) - 1
            back.append(prev)
    return _graph(LAT, E, H, dtype, seed, op, ch, hx)


def _childsums(E, H, dtype, n, depth, wide, seed):
    """Child-sum spines: every level has the level below and some leaves as
    children, `wide` of them at the bottom."""
    rng = np.random.default_rng(seed)
    op, ch, hx = [], [], []
    for _ in range(n):
        top = None
        for d in range(depth):
            kids = [] if top is None else [top]
            for _ in range(wide if d == 0 else int(rng.integers(0, 5))):
                op.append(0), ch.append([]), hx.append(True)
                kids.append(len(op) - 1)
            op.append(1), ch.append(kids), hx.append(False)
            top = len(op) - 1
    return _graph([WL.CS_LEAF, WL.CS_INTERNAL], E, H, dtype, seed, op, ch, hx)


TREE, TREE2 = [WL.NARY_LEAF, WL.NARY_INTERNAL], [WL.NARY_LEAF, WL.NARY_INTERNAL, WL.NARY_INTERNAL]
GRU = [WL.GRU_LEAF, WL.GRU_INTERNAL]
LAT, LGRU = [WL.LAT_CHAR, WL.LAT_WORD], [WL.LGRU_EDGE, WL.POOL_MEAN]
P = functools.partial
# widths: one unit block, a ragged last one, several; rows: one, up to 4 and past 4 per
# team (both forms of the fp32 products), past a tile of 16
CASES = {
    "chain f32 one row": P(_chains, 16, 16, "f32", [9], 1),
    "chain f32 H 20": P(_chains, 12, 20, "f32", [9, 7, 9], 2),
    "chain f32 H 200": P(_chains, 100, 200, "f32", [10, 9, 9, 8, 3, 1, 7], 3),
    "chain f32 H 512": P(_chains, 64, 512, "f32", [8] * 19, 4),
    "chain bf16 H 264": P(_chains, 40, 264, "bf16", [9] * 21, 5),
    "chain bf16 H 24": P(_chains, 8, 24, "bf16", [9, 2, 8], 6),
    "tree f32 H 40": P(_trees, TREE, 28, 40, "f32", 5, 9, 7),
    "tree f32 H 256": P(_trees, TREE, 64, 256, "f32", 23, 9, 8),
    "tree f32 5 rows a team": P(_trees, TREE, 32, 256, "f32", 70, 8, 9),
    "tree f32 19 rows a team": P(_trees, TREE, 32, 256, "f32", 300, 8, 29),
    "tree f32 H 512": P(_trees, TREE, 16, 512, "f32", 3, 8, 10),
    "tree bf16 H 320": P(_trees, TREE, 64, 320, "bf16", 9, 9, 11),
    "tree two types f32": P(_trees, TREE2, 36, 100, "f32", 6, 9, 12),
    "tree two types bf16": P(_trees, TREE2, 40, 104, "bf16", 6, 9, 13),
    "treegru f32 H 72": P(_trees, GRU, 20, 72, "f32", 7, 9, 14),
    "treegru bf16 H 512": P(_trees, GRU, 32, 512, "bf16", 4, 9, 15),
    "grid f32 H 36": P(_grids, 20, 36, "f32", 2, 7, 5, 16),
    "grid bf16 tall": P(_grids, 128, 256, "bf16", 1, 9, 20, 17),
    "grid bf16 H 72": P(_grids, 24, 72, "bf16", 3, 6, 6, 18),
    "lattice f32 H 200": P(_lattices, LAT, 100, 200, "f32", 3, 10, 2, 19),
    "lattice f32 16 words": P(_lattices, LAT, 20, 44, "f32", 2, 10, 16, 20),
    "lattice f32 17 words": P(_lattices, LAT, 20, 44, "f32", 2, 13, 17, 21),
    "lattice bf16 H 88": P(_lattices, LAT, 40, 88, "bf16", 3, 10, 3, 22),
    "lattice f32 characters linked": P(_mixed_lattices, 100, 200, "f32", 3, 10, "char", 32),
    "lattice bf16 characters linked": P(_mixed_lattices, 40, 88, "bf16", 3, 10, "char", 33),
    "lattice f32 word of a word": P(_mixed_lattices, 100, 200, "f32", 3, 10, "word", 34),
    "lattice f32 character after a word": P(_mixed_lattices, 100, 200, "f32", 3, 10, "after", 35),
    "lattice gru f32 H 200": P(_lattices, LGRU, 100, 200, "f32", 3, 9, 2, 23),
    "lattice gru f32 9 edges": P(_lattices, LGRU, 16, 52, "f32", 2, 9, 8, 24),
    "child-sum bf16 H 512": P(_childsums, 64, 512, "bf16", 3, 9, 6, 25),
    "child-sum bf16 32 children": P(_childsums, 32, 96, "bf16", 3, 9, 32, 26),
    "child-sum bf16 33 children": P(_childsums, 32, 96, "bf16", 3, 9, 33, 27),
    "child-sum f32 H 100": P(_childsums, 24, 100, "f32", 5, 9, 8, 28),
}

# more words at one character than a tile holds; links that a lattice's team launch does not
# exchange (only words' c and characters' h travel) up to the last batches; fp32 grids and trees: every batch runs on its own
NO_TEAM = {"lattice f32 17 words", "lattice f32 characters linked", "lattice bf16 characters linked",
           "lattice f32 character after a word", "grid f32 H 36"} | {n for n in CASES if n.startswith("tree") and "f32" in n}


def _teams(f):
    return [f.exec.launch_info(i) for i in range(f.exec.launches())
            if f.exec.launch_info(i)["variant"] == L.TEAM_VARIANT]


@pytest.mark.parametrize("name", sorted(CASES))
def test_team_descriptors_validate(name):
    """The team launch covers a tail of the schedule, and every row, child and
    tile of its descriptors is in range, written once and waited for exactly
    where an earlier tile of the same team writes it."""
    w = CASES[name]()
    for kw in (dict(), dict(plan_mode=L.PLAN_IDENTITY), dict(plan_mode=L.PLAN_PQ)):
        f = edb.Forward(w, flags=L.DRYRUN | L.TEAM_DRYRUN, **kw)
        assert f.exec.validate() >= f.sched.n_batches
        if name in NO_TEAM:
            assert not _teams(f)
            continue
        (t,) = _teams(f)
        B = f.sched.n_batches
        assert t["batch"] + t["n_batches"] == B and t["kind"] == -1 and t["block"] == 512
        assert t["m"] == f.sched.batch_ptr[B] - f.sched.batch_ptr[t["batch"]]
        assert t["grid"] <= 256


def test_team_workloads_validate():
    for k, n in {1: None, 2: None, 3: None, 4: None, 5: 64, 6: None, 7: None, 8: 4, 9: None}.items():
        w = WL.make_config(k, instances=n)
        f = edb.Forward(w, flags=L.DRYRUN | L.TEAM_DRYRUN)
        assert f.exec.validate() >= f.sched.n_batches
        assert bool(_teams(f)) == (k in (1, 3, 5, 9)), k


def test_team_flags():
    """One launch per batch, forced tiles and dry runs keep batches apart."""
    w = WL.make_config(1)
    for fl in (0, L.TEAM_DRYRUN | L.NO_FLOW, L.TEAM_DRYRUN | L.NO_SPLIT_K, L.TEAM_DRYRUN | L.NO_LARGE):
        assert not _teams(edb.Forward(w, flags=L.DRYRUN | fl))
    with pytest.raises(L.EdbError) as ei:
        edb.Forward(w, flags=L.TEAM_DRYRUN)
    assert ei.value.status == L.EDB_ERR_INVALID


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_team_parity(name):
    """Against the oracle (1e-4 fp32, 2e-2 bf16, the library's bounds), on a
    replay too, and bitwise the same through the one-call path and eagerly."""
    torch = pytest.importorskip("torch")
    w = CASES[name]()
    f = edb.Forward(w)
    assert bool(_teams(f)) == (name not in NO_TEAM) and f.exec.validate() >= f.sched.n_batches
    f.run()
    h, c = f.states()
    f.arena_h.fill_(3.0)
    f.arena_c.fill_(float("nan"))
    f.run()
    h2, c2 = f.states()
    np.testing.assert_array_equal(h2, h)
    np.testing.assert_array_equal(c2, c)
    e = edb.Forward(w, flags=L.X_DIRECT | L.FORCE_GATHER)
    e.run()
    h3, c3 = e.states()
    np.testing.assert_array_equal(h3, h)
    np.testing.assert_array_equal(c3, c)
    fc = edb.ForwardCall(w.op_type, w.child_ptr, w.child_idx, w.x_row, w.n_types, edb.operand_shapes(w), f.cells,
                         table=edb.LATTICE_TABLE if w.kinds == LAT else None)
    f.arena_h.fill_(5.0)
    fc.call([b.data_ptr() for b in f.weights], f.x.data_ptr(), f.arena_h.data_ptr(), f.arena_c.data_ptr(),
            f.arena_h.shape[0], f.stream.cuda_stream)
    h4, _ = f.states()
    np.testing.assert_array_equal(h4, h)
    torch.cuda.synchronize()
    err = state_rel_err(h, c, *evaluate_workload(w))
    print(f"team {name}: err {err:.3e}", flush=True)
    assert err <= (1e-4 if w.dtype == "f32" else 2e-2)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_team_nan_states(dtype):
    """Inputs with NaN (the all-ones pattern that marks an empty row among
    them) and infinities: no wait is confused, and the states are NaN exactly
    where one launch per batch makes them NaN."""
    torch = pytest.importorskip("torch")
    w = _chains(16, 48, dtype, [10, 9, 8, 8, 7], 30)
    out = []
    for fl in (L.USE_GRAPH, L.USE_GRAPH | L.NO_FLOW):
        f = edb.Forward(w, flags=fl)
        f.x[3, :] = float("nan")
        f.x[12, 5] = float("inf")
        bits = f.x.view(torch.int32 if dtype == "f32" else torch.int16)
        bits[21, :] = -1
        f.run()
        out.append(f.states())
    for a, b in zip(*out):
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b))
        ok = ~np.isnan(a)
        np.testing.assert_allclose(a[ok], b[ok], rtol=2e-2 if dtype == "bf16" else 1e-4, atol=1e-2 if dtype == "bf16" else 1e-6)


def _dispatch(launches, seed, attend, late=0.0):
    """Model of the device: launches of (P, C) in flight together, their
    work-groups dealt to 8 XCDs of 32 CUs in turn, one to a CU, an XCD's queues
    served in random order; `late` is the share of XCD 7's time lost to earlier
    work.  A work-group takes the launch's next ticket; members of a full team
    run for a while and end; one of an incomplete team holds its CU, with
    `attend` for so many steps at most, then the team is left and its last
    member runs alone.  Returns whether every launch ends, and how many teams
    were left."""
    rng = np.random.default_rng(seed)
    queue = [[[x for x in range(P * C) if x % 8 == xcd] for xcd in range(8)] for P, C in launches]
    ticket, cus = [0] * len(launches), [[] for _ in range(8)]      # (launch, team, end, started)
    left, step = set(), 0
    while any(any(q) for q in queue) or any(cus):
        step += 1
        if step > 4000:
            return False, len(left)
        for xcd in range(8):
            room = 32 - len(cus[xcd])
            if xcd == 7 and rng.random() < late:
                room = 0
            while room and any(q[xcd] for q in queue):
                n = rng.choice([i for i, q in enumerate(queue) if q[xcd]])
                queue[n][xcd].pop()
                P, t = launches[n][0], ticket[n]
                ticket[n] += 1
                cus[xcd].append([n, t // P, None, step])
                room -= 1
        for xcd in range(8):
            keep = []
            for wg in cus[xcd]:
                n, team, end, began = wg
                P = launches[n][0]
                full = ticket[n] >= (team + 1) * P
                if end is None and (n, team) in left:
                    if not full or began < max(w[3] for c in cus for w in c if w[:2] == [n, team]):
                        continue                               # it has left
                    wg[2] = step + 20                          # the last one, alone
                elif end is None and full:
                    wg[2] = step + 5
                elif end is None and attend is not None and step - began > attend:
                    left.add((n, team))
                    continue
                if wg[2] is None or wg[2] > step:
                    keep.append(wg)
            cus[xcd] = keep
    return True, len(left)


def test_team_launches_always_end():
    """Launches that together may hold an XCD's 32 CUs with incomplete teams do
    not stop: a left team's last member walks it alone.  (Members that waited for
    each other without end did stop.)  What the host lets into flight at once, at
    most 31 work-groups of incomplete teams, never comes to that."""
    stopped = 0
    for P, C, n in ((16, 16, 4), (13, 19, 4), (32, 8, 3)):
        for seed in range(12):
            late = (0.0, 0.9, 0.99)[seed % 3]
            stopped += not _dispatch([(P, C)] * n, seed, None, late)[0]
            ends, _ = _dispatch([(P, C)] * n, seed, 300, late)
            assert ends, (P, C, n, seed)
    assert stopped
    for flight in ([(8, 32)] * 4, [(4, 64)] * 4, [(16, 16)] * 2, [(13, 19), (8, 32), (4, 64)], [(32, 8)]):
        for seed in range(12):
            ends, left = _dispatch(flight, seed, None, (0.0, 0.9, 0.99)[seed % 3])
            assert ends and left == 0, (flight, seed)


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(set(CASES) - NO_TEAM))
def test_team_walked_alone(name, monkeypatch):
    """Every team left by its members and walked by the last one alone, and with
    no time given to wait for it some or none: the same states bit for bit,
    eagerly, through the kept sequence and through the one-call path, and no
    wait times out."""
    torch = pytest.importorskip("torch")
    w = CASES[name]()
    f = edb.Forward(w)
    f.run()
    h, c = f.states()
    for flags, spin in ((0, "-1"), (L.USE_GRAPH, "-1"), (0, "0")):
        monkeypatch.setenv("EDB_SPIN_US", spin)
        g = edb.Forward(w, flags=flags)
        assert _teams(g)
        for _ in range(2):
            g.arena_h.fill_(7.0)
            g.arena_c.fill_(-7.0)
            g.run()
            h2, c2 = g.states()
            np.testing.assert_array_equal(h2, h)
            np.testing.assert_array_equal(c2, c)
    fc = edb.ForwardCall(w.op_type, w.child_ptr, w.child_idx, w.x_row, w.n_types, edb.operand_shapes(w), f.cells,
                         table=edb.LATTICE_TABLE if w.kinds == LAT else None)
    f.arena_h.fill_(5.0)
    monkeypatch.setenv("EDB_SPIN_US", "-1")
    fc.call([b.data_ptr() for b in f.weights], f.x.data_ptr(), f.arena_h.data_ptr(), f.arena_c.data_ptr(),
            f.arena_h.shape[0], f.stream.cuda_stream)
    h3, c3 = f.states()
    np.testing.assert_array_equal(h3, h)
    np.testing.assert_array_equal(c3, c)
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_team_wait_bound_is_reported(monkeypatch):
    """Waits that give up at their first look (13 work-groups over 12 steps cannot
    all find their rows written): the launch ends, edb_exec_check reports it, and
    without it the next call of any kind does, once; what runs then is right."""
    torch = pytest.importorskip("torch")
    w = _chains(100, 200, "f32", [12] * 6, 31)
    ok = edb.Forward(w)
    ok.run()
    h, c = ok.states()
    monkeypatch.setenv("EDB_TEAM_RELOADS", "0")
    f = edb.Forward(w, flags=0)
    fc = edb.ForwardCall(w.op_type, w.child_ptr, w.child_idx, w.x_row, w.n_types, edb.operand_shapes(w), f.cells)
    args = ([b.data_ptr() for b in f.weights], f.x.data_ptr(), f.arena_h.data_ptr(), f.arena_c.data_ptr(),
            f.arena_h.shape[0], f.stream.cuda_stream)

    def reported(call):
        torch.cuda.synchronize()
        with pytest.raises(L.EdbError) as ei:
            call()
        assert ei.value.status == L.EDB_ERR_HIP and ("timed out" in str(ei.value) or "its bound" in str(ei.value))

    f.run()
    reported(lambda: f.exec.check(f.stream.cuda_stream))
    f.run()                                   # told already
    reported(lambda: fc.call(*args))          # the next call of another kind
    fc.call(*args)
    reported(lambda: fc.call_noalloc(*args))
    fc.call_noalloc(*args)
    reported(ok.run)
    monkeypatch.delenv("EDB_TEAM_RELOADS")
    ok.arena_h.fill_(9.0)
    ok.run()
    h2, c2 = ok.states()
    np.testing.assert_array_equal(h2, h)
    np.testing.assert_array_equal(c2, c)
    fc.call_noalloc(*args)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(f.arena_h.cpu().numpy()[f.plan.slot], h)
    np.testing.assert_array_equal(f.arena_c.cpu().numpy()[f.plan.slot], c)


@pytest.mark.gpu
def test_captured_stream_is_refused():
    """edb_execute on a stream under capture, its descriptors long uploaded: an
    error, and neither the capture nor later team launches anywhere are harmed."""
    torch = pytest.importorskip("torch")
    w = _chains(16, 48, "bf16", [10, 9, 8, 8, 7], 45)
    f, g = edb.Forward(w), edb.Forward(w, flags=0)
    for e in (f, g):
        assert _teams(e)
        e.run()
    h, c = f.states()
    y = torch.zeros(64, device="cuda")
    graph, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    args = ([b.data_ptr() for b in f.weights], f.x.data_ptr(), f.arena_h.data_ptr(), f.arena_c.data_ptr())
    with torch.cuda.graph(graph, stream=st, capture_error_mode="thread_local"):
        y += 1
        for e in (f, g):
            with pytest.raises(L.EdbError) as ei:
                e.exec.execute(*args, st.cuda_stream)
            assert ei.value.status == L.EDB_ERR_HIP and "captured" in str(ei.value)
        y += 1
    for n in range(1, 4):
        graph.replay()
        for e in (f, g):
            e.arena_h.fill_(4.0)
            e.run()
            h2, c2 = e.states()
            np.testing.assert_array_equal(h2, h)
            np.testing.assert_array_equal(c2, c)
        assert bool((y == 2 * n).all())
    for _ in range(6):       # past every place of the gate
        g.run()
    h2, _ = g.states()
    np.testing.assert_array_equal(h2, h)


@pytest.mark.gpu
def test_team_launches_on_many_streams():
    """Sixteen threads with a stream each run team launches of different
    workloads at once, executors and one-call paths in turn: no wait times
    out (few team launches are in flight at a time) and every arena is
    bitwise the single run's."""
    torch = pytest.importorskip("torch")
    import threading
    ws = [_lattices(LAT, 100, 200, "f32", 24, 12, 2, 40), _chains(64, 256, "bf16", [12] * 40, 41),
          _childsums(64, 512, "bf16", 24, 8, 4, 42), _lattices(LGRU, 100, 200, "f32", 20, 10, 2, 43)]
    ref = []
    for w in ws:
        f = edb.Forward(w)
        assert _teams(f)
        f.run()
        ref.append(f.states())
    streams = [torch.cuda.Stream() for _ in range(16)]
    fs, calls = [], []
    for i, st in enumerate(streams):
        w = ws[i % 4]
        with torch.cuda.stream(st):
            fs.append(edb.Forward(w, flags=L.USE_GRAPH if i % 8 < 4 else 0))
        calls.append(edb.ForwardCall(w.op_type, w.child_ptr, w.child_idx, w.x_row, w.n_types, edb.operand_shapes(w),
                                     fs[i].cells, table=edb.LATTICE_TABLE if w.kinds == LAT else None))
    torch.cuda.synchronize()
    errors = []

    def work(i):
        f = fs[i]
        try:
            for r in range(12):
                if r % 3 == 2:
                    calls[i].call([b.data_ptr() for b in f.weights], f.x.data_ptr(), f.arena_h.data_ptr(),
                                  f.arena_c.data_ptr(), f.arena_h.shape[0], f.stream.cuda_stream)
                else:
                    f.run()
        except Exception as ex:
            errors.append(ex)

    th = [threading.Thread(target=work, args=(i,)) for i in range(16)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errors, errors
    for i, f in enumerate(fs):
        h, c = f.states()
        np.testing.assert_array_equal(h, ref[i % 4][0], err_msg=f"stream {i}")
        np.testing.assert_array_equal(c, ref[i % 4][1], err_msg=f"stream {i}")
    for st in streams:
        edb.ForwardCall.release_stream(st.cuda_stream)


@pytest.mark.gpu
def test_team_launches_on_per_thread_streams():
    """hipStreamPerThread is one handle for a stream of every thread: eight
    threads run team launches through it, and free executors while the others
    run.  Every arena is bitwise the single run's, no wait times out."""
    torch = pytest.importorskip("torch")
    import threading
    w = _chains(64, 256, "bf16", [12] * 40, 44)
    ref = edb.Forward(w)
    assert _teams(ref)
    ref.run()
    h, c = ref.states()
    fs = [[edb.Forward(w, flags=0) for _ in range(3)] for _ in range(8)]
    torch.cuda.synchronize()
    errors = []

    def work(mine):
        try:
            for r in range(9):
                f = mine[r % 3]
                f.exec.execute([b.data_ptr() for b in f.weights], f.x.data_ptr(), f.arena_h.data_ptr(),
                               f.arena_c.data_ptr(), 2)
            for f in mine[:2]:
                f.exec = None          # freed behind its launches
            mine[2].exec.check(2)      # this thread's stream
        except Exception as ex:
            errors.append(ex)

    th = [threading.Thread(target=work, args=(q,)) for q in fs]
    for t in th:
        t.start()
    for t in th:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    s = ref.plan.slot
    for f in sum(fs, []):
        np.testing.assert_array_equal(f.arena_h.float().cpu().numpy()[s], h)
        np.testing.assert_array_equal(f.arena_c.cpu().numpy()[s], c)
