"""Short 1-D grids, whose steps run in one kernel (64 lanes advance a segment
of 52 cells with six halo lanes on each side): the exact build equals the
FP64 oracle bit for bit at sizes around the segment's edges and at the
longest grid that takes the kernel, for every face kind and variant; FP32
equals the two stage kernels (which per-step timing selects) bit for bit;
calls that are split, run past their end or stop at t_stop give the same
state."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 6, 46, 51, 52, 53, 58, 104, 105, 833, 1664, 1665, 2304, 2305]


def _grid(prob, prec, **kw):
    from paper_1607_01105_amd.ppml import Grid

    print(f"[case] {prob.name} n={prob.n[0]} {prec} {kw}", flush=True)
    return Grid.from_problem(prob, prec=prec, exact=True, **kw)


def _problem(n, kind, seed=0):
    p = W.blocks(1, (n,), seed=n + seed)
    if kind == "inflow":
        p.bc = [("inflow", "outflow")] + p.bc[1:]
        p.inflow = {0: (1.4, 0.7, 0.0, 0.0, 1.0)}
    elif kind == "inflow_hi":
        p.bc = [("reflect", "inflow")] + p.bc[1:]
        p.inflow = {1: (0.6, -0.4, 0.0, 0.0, 0.8)}
    elif kind == "walls":
        p.bc = [("reflect", "outflow")] + p.bc[1:]
    elif kind != "periodic":
        p.bc = [(kind, kind)] + p.bc[1:]
    return p


def _equal_oracle(g, o, steps, taus):
    t, dt, taken = g.time()
    assert taken == steps and t == o.t and dt == taus[-1]
    for f in (0, 1, 4, 5):
        assert np.array_equal(g.get(f), o.get(f)), f
    assert g.max_speeds() == o.max_speeds()


@pytest.mark.parametrize("kind", ["periodic", "outflow", "walls", "inflow", "inflow_hi"])
@pytest.mark.parametrize("n", SIZES)
def test_exact_fp64_equals_oracle(n, kind):
    if n < 3 and kind in ("walls", "inflow_hi"):
        pytest.skip("a reflecting axis needs three cells")
    prob = _problem(n, kind)
    steps = 7 if n > 1000 else 33
    o = make_oracle(prob)
    taus = o.run(steps)
    g = _grid(prob, "fp64")
    g.step(3)
    g.step(steps - 3)
    _equal_oracle(g, o, steps, taus)


@pytest.mark.parametrize("variant", ["first_order", "isothermal", "uniform", "log"])
def test_variants_equal_oracle(variant):
    prob = _problem(157, "walls")
    kw = {}
    if variant == "first_order":
        kw["first_order"] = True
    elif variant == "isothermal":
        prob.isothermal = 0.8
        prob.p = 0.64 * prob.rho
    elif variant == "uniform":
        prob.potential = ("uniform", 0.3, 0.0, 0.0)
    else:
        prob.potential = ("log", 0.5, 0.2, 1.0, 0.4, 0.0, 0.0)
    o = make_oracle(prob, first_order=variant == "first_order")
    taus = o.run(20)
    g = _grid(prob, "fp64", **kw)
    g.step(20)
    _equal_oracle(g, o, 20, taus)


@pytest.mark.parametrize("n", [5, 52, 105, 1024, 3840, 3841])
@pytest.mark.parametrize("kind", ["periodic", "walls", "inflow"])
def test_exact_fp32_equals_stage_kernels(n, kind):
    import torch

    prob = _problem(n, kind)
    a, b = _grid(prob, "fp32"), _grid(prob, "fp32")
    b.set_timing(20)
    a.step(25)
    b.step(25)  # 20 timed steps through the stage kernels, the rest through the line kernel
    assert a.time() == b.time() and a.max_speeds() == b.max_speeds()
    assert torch.equal(a.state, b.state)


def test_split_calls_and_t_stop():
    import torch

    prob = _problem(200, "outflow")
    a, b = _grid(prob, "fp64"), _grid(prob, "fp64")
    a.step(1500)  # more steps than one launch takes
    for _ in range(5):
        b.step(300)
    assert a.time() == b.time() and torch.equal(a.state, b.state)
    o = make_oracle(prob)
    taus = o.run(100, t_stop=0.05)
    c = _grid(prob, "fp64")
    c.step(100, t_stop=0.05)
    c.step(5, t_stop=0.05)  # past the end: no step
    _equal_oracle(c, o, len(taus), taus)
    fixed = _grid(prob, "fp64")
    o = make_oracle(prob)
    taus = o.run(9, dt_fixed=1e-4)
    fixed.step(9, dt_fixed=1e-4)
    _equal_oracle(fixed, o, 9, taus)
