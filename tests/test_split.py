"""The split tile: fp32 batches through three bf16 pieces per operand."""
import dataclasses

import numpy as np
import pytest

from oracle.compare import state_rel_err
from oracle.evaluate import evaluate_workload
from paper_2302_03851_amd import _lib as L
from paper_2302_03851_amd import edb
from paper_2302_03851_amd import workloads as WL

TREE, GRU = [WL.NARY_LEAF, WL.NARY_INTERNAL], [WL.GRU_LEAF, WL.GRU_INTERNAL]


def _pairs(kinds, E, H, n, seed, scale=0.1):
    """n trees of two leaves (every third with an absent right child)."""
    op, ch, hx = [], [], []
    for t in range(n):
        k = len(op)
        op += [0, 0, 1]
        ch += [[], [], [k, k + 1 if t % 3 else -1]]
        hx += [True, True, False]
    return WL.make_graph(kinds, E, H, op, ch, hx, seed=seed, scale=scale, bias_scale=0.2)


def _chains(E, H, n, seed):
    op, ch = [0] * (3 * n), [[-1] if i % 3 == 0 else [i - 1] for i in range(3 * n)]
    return WL.make_graph([WL.LSTM_CHAIN], E, H, op, ch, [True] * (3 * n), seed=seed, bias_scale=0.2)


def _config(k, instances, E, H):
    """A configuration's graphs with dimensions of whole groups of 32."""
    w, rng = WL.make_config(k, instances=instances), np.random.default_rng(k)
    weights = [{n: np.eye(H, dtype=np.float32) if kind == WL.POOL_MEAN and len(s) == 2 and s[0] == s[1] else
                rng.uniform(-0.1, 0.1, size=s).astype(np.float32)
                for n, s in WL.weight_shapes(kind, E, H, w.n_children[t] or 2)} for t, kind in enumerate(w.kinds)]
    x = rng.standard_normal(size=(w.x.shape[0], E), dtype=np.float32)
    return dataclasses.replace(w, in_dim=E, hidden=H, weights=weights, x=x)


# rows: under, at and past a tile of 64 and of 32; E and H of whole and of padded groups of 32
CASES = [(_pairs, TREE, 64, 128, 31, 1), (_pairs, TREE, 24, 92, 65, 2), (_pairs, GRU, 32, 64, 64, 3),
         (_pairs, GRU, 56, 188, 33, 4), (_chains, 60, 124, 97, 5),
         (_pairs, [WL.CS_LEAF, WL.CS_INTERNAL], 64, 64, 20, 6), (_config, 3, 2, 96, 188),
         (_config, 9, 2, 60, 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("variant", L.SPLIT_VARIANTS)
@pytest.mark.parametrize("case", range(len(CASES)))
def test_split_tile_precision(case, variant, monkeypatch):
    """Forced onto every batch: within the library's fp32 bound of the oracle,
    and no further from it than one launch of fp32 products per batch."""
    pytest.importorskip("torch")
    make, *args = CASES[case]
    w = make(*args)
    ref = evaluate_workload(w)
    err = []
    for v in (16, variant):
        monkeypatch.setenv("EDB_VARIANT", str(v))
        f = edb.Forward(w)
        used = {f.exec.launch_info(i)["variant"] for i in range(1, f.exec.launches())}
        assert v in used, used
        f.run()
        h, c = f.states()
        err.append((state_rel_err(h, c, *ref), np.sqrt(np.sum((h - ref[0]) ** 2) + np.sum((c - ref[1]) ** 2))))
    print(f"split variant {variant} case {case}: max {err[1][0]:.2e}, 2-norm {err[1][1]:.3e}, fp32 products "
          f"{err[0][1]:.3e}", flush=True)
    assert err[1][0] <= 1e-4 and err[1][1] <= err[0][1]


@pytest.mark.gpu
@pytest.mark.parametrize("nonzero", [1, 2, 4, 16, 64])
@pytest.mark.parametrize("kinds", [TREE, GRU, [WL.LSTM_CHAIN]])
def test_split_tile_sparse_rows(kinds, nonzero, monkeypatch):
    """Rows of x with few non-zeros (one-hot, masked), without biases: no
    further from the oracle than fp32 products.  With one non-zero both round
    once and the pieces leave out another sixth of that (1.5% of a 2-norm);
    the norms of 3,840 states differ by 2% from sample to sample: 1.05."""
    pytest.importorskip("torch")
    if kinds == [WL.LSTM_CHAIN]:
        w = _chains(512, 64, 20, 11)
        for n in w.weights[0]:
            w.weights[0][n] *= 5.0
    else:
        w = _pairs(kinds, 512, 64, 100, 11, scale=0.5)
    rng = np.random.default_rng(nonzero)
    for row in w.x:
        row[rng.permutation(512)[nonzero:]] = 0.0
    for d in w.weights:
        for n in d:
            if n.startswith("b"):
                d[n][:] = 0.0
    ref = evaluate_workload(w)
    err = []
    for v in (16,) + L.SPLIT_VARIANTS:
        monkeypatch.setenv("EDB_VARIANT", str(v))
        f = edb.Forward(w)
        f.run()
        h, c = f.states()
        err.append(np.sqrt(np.sum((h - ref[0]) ** 2) + np.sum((c - ref[1]) ** 2)))
    print(f"split kinds {kinds} nonzero {nonzero}: fp32 {err[0]:.3e}, split {err[1]:.3e} {err[2]:.3e} {err[3]:.3e}", flush=True)
    assert max(err[1:]) <= 1.05 * err[0]


@pytest.mark.gpu
def test_split_tile_chosen_and_bitwise_across_layouts():
    """The default for large fp32 batches; layouts and launch modes agree
    bitwise, and EDB_NO_SPLIT_K and EDB_TILE_LARGE keep to fp32 products."""
    pytest.importorskip("torch")
    w = _pairs(TREE, 64, 256, 4000, 6)
    f = edb.Forward(w)
    kinds = [f.exec.launch_info(i)["variant"] for i in range(1, f.exec.launches())]
    assert any(v in L.SPLIT_VARIANTS for v in kinds), kinds
    f.run()
    h, c = f.states()
    for kw in (dict(flags=0), dict(plan_mode=L.PLAN_IDENTITY), dict(flags=L.USE_GRAPH | L.FORCE_GATHER | L.X_DIRECT)):
        g = edb.Forward(w, **kw)
        g.run()
        h2, c2 = g.states()
        np.testing.assert_array_equal(h2, h)
        np.testing.assert_array_equal(c2, c)
    for fl in (L.NO_SPLIT_K, L.TILE_LARGE, L.NO_LARGE):
        g = edb.Forward(w, flags=fl)
        assert not any(g.exec.launch_info(i)["variant"] in L.SPLIT_VARIANTS for i in range(1, g.exec.launches()))


@pytest.mark.gpu
def test_split_tile_not_finite(monkeypatch):
    """Infinities, NaN and values near the ends of the fp32 range in x: the
    states are finite and NaN where the fp32 products make them so."""
    pytest.importorskip("torch")
    w = _pairs(TREE, 64, 64, 40, 7)
    out = []
    for v in (16, L.SPLIT_VARIANTS[0]):
        monkeypatch.setenv("EDB_VARIANT", str(v))
        f = edb.Forward(w)
        f.x[0, 3], f.x[5, 7], f.x[9, 1] = float("inf"), float("-inf"), float("nan")
        f.x[12, :], f.x[20, :], f.x[30, :] = 1e38, 3e-39, -2e-30
        f.run()
        out.append(f.states())
    for a, b in zip(*out):
        np.testing.assert_array_equal(np.isnan(a), np.isnan(b))
        ok = ~np.isnan(a)
        np.testing.assert_allclose(a[ok], b[ok], rtol=1e-4, atol=1e-6)


def _two_levels(E, H, n):
    """n trees of two internal nodes, one above the other: two batches of n rows."""
    op, ch, hx = [], [], []
    for t in range(n):
        k = len(op)
        op += [0, 0, 0, 1, 1]
        ch += [[], [], [], [k, k + 1], [k + 3, k + 2]]
        hx += [True, True, True, False, False]
    return WL.make_graph(TREE, E, H, op, ch, hx, seed=12)


def test_split_class_does_not_depend_on_the_batch_order():
    """The first batch of a type, which pays for the weights' splitting, takes
    the class that a later one of the same rows takes."""
    used = set()
    for H in (192, 320, 512, 768, 1024):
        for n in (180, 260, 380, 550, 800, 1100, 1300, 1600, 2000, 3200, 5000):
            f = edb.Forward(_two_levels(64, H, n), flags=L.DRYRUN | L.TEAM_DRYRUN)
            got = [q["variant"] for q in (f.exec.launch_info(i) for i in range(1, f.exec.launches()))
                   if q["kind"] == WL.NARY_INTERNAL]
            assert len(got) == 2
            if got[0] in L.SPLIT_VARIANTS:
                assert got[0] == got[1], (H, n, got)
                used.add(got[0])
    assert used == set(L.SPLIT_VARIANTS)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", L.SPLIT_VARIANTS)
def test_split_tile_ends_of_the_range(variant, monkeypatch):
    """The lowest and the largest fp32 value, which no bf16 value reaches, on a
    zero weight and beside each other on weights that leave a finite sum (every
    gate saturates upwards): finite states, the fp32 products'."""
    pytest.importorskip("torch")
    low, top = float(np.finfo(np.float32).min), float(np.finfo(np.float32).max)
    w = _pairs(TREE, 64, 64, 40, 9)
    W = w.weights[0]["W"]
    W[3, :], W[8, :], W[9, :] = 0.0, -0.05, 0.03
    out = []
    for v in (16, variant):
        monkeypatch.setenv("EDB_VARIANT", str(v))
        f = edb.Forward(w)
        f.x[0, 3] = f.x[1, 3] = low
        f.x[2, 3] = top
        f.x[6, 8] = f.x[6, 9] = low
        f.x[7, 8], f.x[9, 9], f.x[10, 9] = low, top, 3.396e38
        f.run()
        out.append(f.states())
    for a, b in zip(*out):
        assert np.isfinite(a).all()
        np.testing.assert_allclose(b, a, rtol=1e-4, atol=1e-6)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", L.SPLIT_VARIANTS)
def test_split_tile_infinite_weights(variant, monkeypatch):
    """Infinite, NaN and the largest weights, of the leaves (x, infinite among
    it) and of their parents (h): NaN where the fp32 products are, the same
    states elsewhere."""
    pytest.importorskip("torch")
    inf, top = float("inf"), float(np.finfo(np.float32).max)
    w = _pairs(TREE, 64, 64, 40, 10)
    W, U = w.weights[0]["W"], w.weights[1]["W"]
    W[5, 70:80], W[6, 150:160], W[7, 3], W[9, 130], W[10, 20] = inf, -inf, float("nan"), top, -300.7
    U[3, 5], U[80, 200], U[100, 9], U[101, 10] = inf, -inf, top, -top
    out = []
    for v in (16, variant):
        monkeypatch.setenv("EDB_VARIANT", str(v))
        f = edb.Forward(w)
        f.x[:, 5:12] = f.x[:, 5:12].abs() + 0.1   # the leaves' saturated gates are open, their tanh is 1
        f.x[:, 6] *= -1
        f.x[4, 5], f.x[8, 6], f.x[12, 10], f.x[16, 30] = 0.0, inf, -inf, inf
        f.run()
        out.append(f.states())
    for a, b in zip(*out):
        assert np.isnan(a).any() and np.isfinite(a).sum() > a.size // 4
        np.testing.assert_array_equal(np.isnan(b), np.isnan(a))
        ok = ~np.isnan(a)
        np.testing.assert_allclose(b[ok], a[ok], rtol=1e-4, atol=1e-6)


@pytest.mark.gpu
def test_noalloc_fits_without_the_pieces():
    """Trees whose weights' pieces (63 MB) exceed the allocation-free call's
    fixed array: the call still runs, on fp32 products; the default forward
    uses the split tile (both within 1e-5 of each other, states below 1)."""
    torch = pytest.importorskip("torch")
    w = _pairs(TREE, 32, 1024, 1024, 8, scale=0.02)
    f = edb.Forward(w)
    assert any(f.exec.launch_info(i)["variant"] in L.SPLIT_VARIANTS for i in range(1, f.exec.launches()))
    f.run()
    h, c = f.states()
    fc = edb.ForwardCall(w.op_type, w.child_ptr, w.child_idx, w.x_row, w.n_types, edb.operand_shapes(w), f.cells)
    ah, ac = torch.full_like(f.arena_h, 7.0), torch.full_like(f.arena_c, 7.0)
    fc.call_noalloc([b.data_ptr() for b in f.weights], f.x.data_ptr(), ah.data_ptr(), ac.data_ptr(), ah.shape[0],
                    f.stream.cuda_stream)
    torch.cuda.synchronize()
    s = f.plan.slot
    np.testing.assert_allclose(ah.cpu().numpy()[s], h, rtol=1e-5, atol=1e-5)
    np.testing.assert_allclose(ac.cpu().numpy()[s], c, rtol=1e-5, atol=1e-5)
