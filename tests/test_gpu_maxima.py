"""CFL maxima of a state, spread over slots whose number follows the grid's
size: after a set and after steps they are, bit for bit, the maxima over the
cells of the state read back (exact build: the same IEEE operations), at
sizes on both sides of a change of the slot count and at its cap."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(1,), (255,), (4096,), (21846,), (64, 64), (256, 256), (257, 200), (31, 33, 35), (96, 100, 104)]


def _cell_maxima(g, gamma):
    r, mx, my, mz, _, e = g.conserved()
    u = [m / r for m in (mx, my, mz)]
    v = np.sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2])
    c = np.sqrt(gamma * ((gamma - 1.0) * e) / r)
    return float(v.max()), float(c.max())


@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_maxima_equal_the_cells_maxima(n):
    from paper_1607_01105_amd import workloads as W
    from paper_1607_01105_amd.ppml import Grid

    prob = W.random_smooth(len(n), n, seed=sum(n))
    g = Grid.from_problem(prob, prec="fp64", exact=True)
    assert g.max_speeds() == _cell_maxima(g, prob.gamma)
    for steps in (1, 2, 33):
        g.step(steps)
        g.sync()
        assert g.max_speeds() == _cell_maxima(g, prob.gamma), steps
