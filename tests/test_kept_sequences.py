"""EDB_USE_GRAPH: a short sequence is kept as a list of calls, a long one as a HIP graph."""
import numpy as np
import pytest

from paper_2302_03851_amd import _lib as L
from paper_2302_03851_amd import edb
from paper_2302_03851_amd import workloads as WL


def _chain(n, seed):
    """A chain of n nodes: n launches under EDB_NO_FLOW (staging folded or not, + 1)."""
    return WL.make_graph([WL.LSTM_CHAIN], 32, 32, [0] * n, [[-1]] + [[i] for i in range(n - 1)], [True] * n, seed=seed)


@pytest.mark.gpu
@pytest.mark.parametrize("nodes", [1, 2, 30, 31, 32, 33, 40])
def test_kept_sequence_replays_equal_eager(nodes):
    """Either side of 32 calls: executors of the same sequence run in turn on one
    stream, with eager work and synchronisations between their replays, each
    equal to its eager execution; new inputs update the kept sequence."""
    torch = pytest.importorskip("torch")
    flags = L.NO_FLOW
    ws = [_chain(nodes, s) for s in (1, 2)]
    ref = []
    for w in ws:
        f = edb.Forward(w, flags=flags)
        f.run()
        ref.append(f.states())
    # one executor each, on one stream: they share the kept sequence
    with torch.cuda.stream(torch.cuda.Stream()):
        fs = [edb.Forward(w, flags=flags | L.USE_GRAPH) for w in ws]
    fs[0].run()
    i0, u0 = edb.graph_stats()
    for rep in range(4):
        for f, (h, c) in zip(fs, ref):
            f.arena_h.fill_(3.0)
            f.arena_c.fill_(-3.0)
            torch.cuda.synchronize()
            f.run()
            h2, c2 = f.states()
            np.testing.assert_array_equal(h2, h)
            np.testing.assert_array_equal(c2, c)
            f.run()                       # a second time with the same arguments
            h2, c2 = f.states()
            np.testing.assert_array_equal(h2, h)
            np.testing.assert_array_equal(c2, c)
    i1, u1 = edb.graph_stats()
    assert (i1 - i0, u1 - u0) == (0, 7)
