"""An MV-RNN vector batch in one launch (cells of up to 64 units)."""
import numpy as np
import pytest

from paper_2302_03851_amd import _lib as L
from paper_2302_03851_amd import edb
from paper_2302_03851_amd import workloads as WL

MV_VARIANT = 21


def _mv_trees(d, n, seed):
    """n trees of two and of three leaves in turn: a vector and d matrix columns a node."""
    op, ch, hx = [], [], []

    def leaf():
        first = len(op)
        for _ in range(d + 1):
            op.append(0); ch.append([]); hx.append(True)
        return first + d, first

    def parent(l, r):
        first = len(op)
        for j in range(d):
            op.append(1); ch.append([l[1] + j, r[1] + j]); hx.append(False)
        op.append(2)
        ch.append([l[0], r[0]] + [l[1] + j for j in range(d)] + [r[1] + j for j in range(d)])
        hx.append(False)
        return first + d, first

    for t in range(n):
        top = parent(leaf(), leaf())
        if t % 2:
            parent(top, leaf())
    return WL.make_graph([WL.LINEAR, WL.MV_MAT, WL.MV_VEC], d, d, op, ch, hx, seed=seed, bias_scale=0.2)


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(4, 1), (12, 3), (16, 2), (44, 5), (60, 3), (64, 1), (64, 7), (68, 3)])
def test_mv_vec_launch(d, n):
    """Odd and even row counts, one row, padded and whole reductions: as the two
    launches of EDB_NO_SPLIT_K (their sums of at most 2 d terms in another
    order: 1e-5 of states below 1), bitwise repeatable; wider cells keep two."""
    pytest.importorskip("torch")
    w = _mv_trees(d, n, 3)
    out = []
    for flags in (0, L.NO_SPLIT_K, L.USE_GRAPH, L.FORCE_GATHER):
        f = edb.Forward(w, flags=flags)
        kinds = [f.exec.launch_info(i) for i in range(1, f.exec.launches())]
        one = [q["part"] for q in kinds if q["kind"] == WL.MV_VEC]
        assert set(one) == ({0} if d <= 64 and not flags & L.NO_SPLIT_K else {0, 1})
        assert (d <= 64 and not flags & L.NO_SPLIT_K) == any(q["variant"] == MV_VARIANT for q in kinds)
        f.exec.validate(64)
        f.arena_h.fill_(float("nan"))
        f.arena_c.fill_(float("nan"))
        f.run()
        out.append(f.states())
    for k in (0, 1):
        assert np.isfinite(out[0][k]).all()
        np.testing.assert_allclose(out[0][k], out[1][k], rtol=1e-5, atol=1e-5)
        np.testing.assert_array_equal(out[0][k], out[2][k])
        np.testing.assert_array_equal(out[0][k], out[3][k])
