"""Calls of one to three steps take the line kernel for shorter grids than longer
calls do, alone and in batches: sizes on either side, in calls of changing
length, give the oracle's bits (exact FP64) and those of one call (product)."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

CALLS = (1, 2, 3, 4, 1, 5, 2)
SIZES = {"fp64": (1856, 1857, 2176, 2177, 2304), "fp32": (2752, 2753, 3392, 3393, 3712, 3713, 3840)}


def _state(g, ndim):
    return [g.get(f) for f in (0, *range(1, 1 + ndim), 4, 5)] + [np.array(g.time())]


@pytest.mark.parametrize("exact,prec", [(True, "fp64"), (False, "fp64"), (False, "fp32")],
                         ids=["exact_fp64", "fp64", "fp32"])
def test_changing_call_lengths(exact, prec):
    from paper_1607_01105_amd.ppml import Batch, Grid

    probs = [W.blocks(1, (n,), seed=n, bc="reflect") for n in SIZES[prec]]
    want = []
    for prob in probs:
        print(f"[case] {prob.n[0]} {prec} exact={exact} calls of {CALLS}", flush=True)
        one = Grid.from_problem(prob, prec=prec, exact=exact)
        one.step(sum(CALLS))
        want.append(_state(one, 1))
        if exact:
            o = make_oracle(prob)
            o.run(sum(CALLS))
            for f, x in zip((0, 1, 4, 5), want[-1]):
                assert np.array_equal(x, o.get(f)), (prob.n[0], f)
        g = Grid.from_problem(prob, prec=prec, exact=exact)
        for k in CALLS:
            g.step(k)
        for x, y in zip(_state(g, 1), want[-1]):
            assert np.array_equal(x, y), prob.n[0]
    for graph in (False, True):
        print(f"[case] batch of {SIZES[prec]} {prec} exact={exact} graph={graph}", flush=True)
        b = Batch(len(probs), exact=exact)
        slots = [b.admit(b.new_grid(p, prec=prec)) for p in probs]
        for k in CALLS:
            b.step(k, graph=graph)
        b.sync()
        for s, w in zip(slots, want):
            for x, y in zip(_state(b.grids[s], 1), w):
                assert np.array_equal(x, y)
