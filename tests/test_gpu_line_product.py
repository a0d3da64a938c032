"""Product build, 1-D: the line kernel's bits are those of the stage kernels
(which per-step timing selects), in both precisions and every variant; and grids
too long for the line kernel reach the stage kernels' tile shapes, alone and in
batches: the same bits for every shape, the exact build's against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(n, kind, seed=0):
    p = W.blocks(1, (n,), seed=n + seed)
    if kind == "inflow":
        p.bc = [("inflow", "reflect")] + p.bc[1:]
        p.inflow = {0: (1.4, 0.7, 0.0, 0.0, 1.0)}
    elif kind == "walls":
        p.bc = [("reflect", "outflow")] + p.bc[1:]
    elif kind == "isothermal":
        p.isothermal = 0.8
        p.p = 0.64 * p.rho
    elif kind == "uniform":
        p.potential = ("uniform", 0.3, 0.0, 0.0)
    return p


@pytest.mark.parametrize("kind", ["periodic", "walls", "inflow", "isothermal", "uniform", "first_order"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_line_kernel_equals_stage_kernels(prec, kind):
    import torch

    from paper_1607_01105_amd.ppml import Grid

    for n in (3, 52, 105, 833, 1664, 2304, *((3840,) if prec == "fp32" else ())):
        print(f"[case] product {n} {prec} {kind}", flush=True)
        prob = _problem(n, kind)
        a, b = (Grid.from_problem(prob, prec=prec, first_order=kind == "first_order") for _ in range(2))
        b.set_timing(40)
        a.step(40)
        b.step(40)
        assert a.time() == b.time() and a.max_speeds() == b.max_speeds()
        assert torch.equal(a.state, b.state), n


LONG = {"fp64": (2305, 5003), "fp32": (3841, 5003)}


@pytest.mark.parametrize("exact,prec", [(True, "fp64"), (False, "fp64"), (False, "fp32")],
                         ids=["exact_fp64", "fp64", "fp32"])
def test_tile_shapes_of_long_lines(exact, prec):
    from paper_1607_01105_amd.ppml import Batch, Grid, ppml_tile_count

    beside = W.blocks(2, (40, 30), seed=3)  # a batch with 2-D grids takes lines of up to 4608 cells in memory
    for n in LONG[prec]:
        prob = _problem(n, "walls")
        want = None
        if exact:
            o = make_oracle(prob)
            o.run(9)
            want = [o.get(f) for f in (0, 1, 4, 5)]
        for v in range(ppml_tile_count(1)):
            print(f"[case] {n} {prec} exact={exact} tile={v}", flush=True)
            g = Grid.from_problem(prob, prec=prec, exact=exact, tile=v)
            g.step(9)
            out = [[g.get(f) for f in (0, 1, 4, 5)]]
            for others in ([], [beside]):
                b = Batch(3, exact=exact)
                b.set_tile(1, v)
                slots = [b.admit(b.new_grid(p, prec=prec)) for p in [prob, prob, *others]]
                b.step(9, graph=False)
                b.sync()
                out += [[b.grids[s].get(f) for f in (0, 1, 4, 5)] for s in slots[:2]]
            want = want or out[0]
            for got in out:
                for x, y in zip(got, want):
                    assert np.array_equal(x, y), (n, v)
