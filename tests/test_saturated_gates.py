"""Gates far out on both sides (pre-activations of +-10^4): the cell update's
exponentials overflow and underflow together, and the states are still the
limits, 0 and +-1 times what they multiply."""
import dataclasses

import numpy as np
import pytest

from oracle.compare import state_rel_err
from oracle.evaluate import evaluate_workload
from paper_2302_03851_amd import _lib as L
from paper_2302_03851_amd import edb
from paper_2302_03851_amd import workloads as WL


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [L.USE_GRAPH, L.NO_FLOW | L.NO_SPLIT_K])
@pytest.mark.parametrize("k,n", [(1, 4), (2, 6), (3, 2), (4, 2), (5, 3), (7, 5)])
def test_saturated_gates(k, n, flags):
    """Finite, and the oracle's states.  A sum of up to 512 products of up to
    4 * 10^3 is off by sqrt(512) 4 * 10^3 2^-24 = 5.4e-3 in fp32, which shows
    where a pre-activation happens to lie near 0, and a state by as much: 1e-2
    (bf16 2e-2, the library's bound, its x being exact in both)."""
    pytest.importorskip("torch")
    w = WL.make_config(k, instances=n)
    w = dataclasses.replace(w, x=WL.round_bf16(w.x * 1e4) if w.dtype == "bf16" else w.x * np.float32(1e4))
    f = edb.Forward(w, flags=flags)
    f.run()
    h, c = f.states()
    assert np.isfinite(h).all() and np.isfinite(c).all()
    with np.errstate(over="ignore"):
        ref = evaluate_workload(w)
    assert state_rel_err(h, c, *ref) <= (1e-2 if w.dtype == "f32" else 2e-2)
