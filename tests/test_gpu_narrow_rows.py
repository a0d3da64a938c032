"""Narrow FP64 3-D grids take the row kernels from some hundred rows on, the
marching kernels below: sizes on either side give the oracle's bits."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(8, 21, 24), (8, 16, 32), (9, 10, 12), (3, 20, 26)], ids=lambda n: "x".join(map(str, n)))
def test_narrow_rows(n):
    from paper_1607_01105_amd.ppml import Grid

    prob = W.blocks(3, n, seed=n[2])
    print(f"[case] {n} fp64 exact, 5 steps", flush=True)
    g = Grid.from_problem(prob, prec="fp64", exact=True)
    g.step(5)
    o = make_oracle(prob)
    o.run(5)
    for f in range(6):
        assert np.array_equal(g.get(f), o.get(f)), f
