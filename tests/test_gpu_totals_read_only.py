"""Reads of a grid leave its work area's stage output as it was: another thread's
steps of the batch that holds the grid may be using it."""
from __future__ import annotations

import pytest

from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [(700,), (90, 70), (40, 36, 33)], ids=lambda n: "x".join(map(str, n)))
def test_reads_leave_the_stage_output(n, prec):
    import torch

    from paper_1607_01105_amd.ppml import Grid

    print(f"[case] {n} {prec}", flush=True)
    g = Grid.from_problem(W.blocks(len(n), n, seed=2), prec=prec)
    half = g.scratch[: g.state.numel()]  # the stage output lies first
    half.fill_(0xA5)
    torch.cuda.synchronize()
    totals = g.totals()
    g.max_speeds(), g.time(), g.sync()
    for f in (0, *range(1, 1 + len(n)), 4, 5):
        assert abs(g.get(f).sum() - totals[f]) <= 1e-12 * abs(g.get(f)).sum() + 1e-300
    assert bool((half == 0xA5).all())
