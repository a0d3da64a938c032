"""A grid on hipStreamPerThread, which is another stream in every thread: set and
get calls of several chunks are ordered with the steps that the calling thread
has queued (the bits of the same calls on an ordinary stream)."""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import pytest

from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

PER_THREAD = SimpleNamespace(cuda_stream=2)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("prob", [W.blocks(2, (700, 500), seed=5), W.periodic_modes(80, seed=3)], ids=["2d", "3d"])
def test_set_and_get_follow_queued_steps(prob, prec):
    import torch

    from paper_1607_01105_amd.ppml import Grid

    print(f"[case] {prob.name} {prec} on the per-thread stream", flush=True)
    fields = [0, *range(1, 1 + prob.ndim), 4, 5]
    a = Grid.from_problem(prob, prec=prec, stream=PER_THREAD)
    b = Grid.from_problem(prob, prec=prec, stream=torch.cuda.Stream())
    for g in (a, b):
        g.step(60)
        g.first = [g.get(f) for f in fields]  # behind the steps, without a wait of its own
        g.step(40)
        g.set_conserved(g.conserved(), rho_mean0=1.0)
        g.step(3)
        g.set_primitive(prob.rho, prob.vx, prob.vy, prob.vz, prob.p)
        g.step(5)
        g.last = [g.get(f) for f in fields]
    for x, y in zip(a.first + a.last, b.first + b.last):
        assert np.array_equal(x, y)
    assert a.time() == b.time()
