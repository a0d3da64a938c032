"""FP64 3-D launches choose between 32x8 and 16x16 tiles for the default shape by
the cells that each takes to cover the grids: grids of both kinds, too large for
the row kernels, give the bits of the shapes named, alone and in batches that
fall on either side."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

NARROW = (64, 24, 100)  # 24 rows: three tiles of 8, two of 16
WIDE = (100, 100, 30)


def _state(g):
    return [g.get(f) for f in range(6)] + [np.array(g.time()[:2])]


@pytest.mark.parametrize("exact", [True, False], ids=["exact", "product"])
def test_default_shape_gives_the_bits_of_the_named_ones(exact):
    from paper_1607_01105_amd.ppml import Batch, Grid, ppml_tile_count

    solo = {}
    for n in (NARROW, WIDE):
        prob = W.blocks(3, n, seed=n[2])
        for v in range(ppml_tile_count(3)):
            print(f"[case] {n} fp64 exact={exact} tile={v}", flush=True)
            g = Grid.from_problem(prob, prec="fp64", exact=exact, tile=v)
            g.step(4)
            out = _state(g)
            for a, b in zip(out, solo.setdefault(n, out)):
                assert np.array_equal(a, b), (n, v)
    for sizes in ([NARROW], [WIDE], [NARROW, NARROW, WIDE], [NARROW, WIDE]):
        print(f"[case] batch {sizes} fp64 exact={exact}", flush=True)
        b = Batch(4, exact=exact)
        slots = [b.admit(b.new_grid(W.blocks(3, n, seed=n[2]), prec="fp64")) for n in sizes]
        b.step(4, graph=False)
        b.sync()
        for n, s in zip(sizes, slots):
            for x, y in zip(_state(b.grids[s]), solo[n]):
                assert np.array_equal(x, y), (sizes, n)
