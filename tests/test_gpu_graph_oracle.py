"""Long ppml_step calls that replay the captured chunk, against the oracle: 2-D,
3-D and 1-D grids past the line kernel's length (shorter ones take all steps of a
call in that kernel), run to t_stop in calls of 64 steps, exact build."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prob,steps", [(W.blocks(1, (2400,), seed=5), 150), (W.blocks(2, (45, 37), seed=8, bc="reflect"), 150),
                                        (W.periodic_modes(24, seed=2), 100), (W.blocks(3, (70, 70, 62), seed=4), 70)],
                         ids=["1d", "2d", "3d_rows", "3d_march"])
def test_replayed_chunks_equal_the_oracle(prob, steps):
    from paper_1607_01105_amd.ppml import Grid

    o = make_oracle(prob)
    taus = o.run(steps)
    t_stop = float(sum(taus[:-1])) + 0.5 * float(taus[-1])  # within the last step
    o = make_oracle(prob)
    taus = o.run(10 ** 6, t_stop=t_stop)
    print(f"[case] {prob.name} exact fp64, {len(taus)} steps in calls of 64", flush=True)
    g = Grid.from_problem(prob, prec="fp64", exact=True)
    t, _, n = g.run_to(t_stop, chunk=64)
    assert t == o.t and n == len(taus)
    for f in (0, *range(1, 1 + prob.ndim), 4, 5):
        assert np.array_equal(g.get(f), o.get(f)), f
