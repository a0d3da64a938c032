"""Small 3-D grids, whose stage kernels give a wave the strip of a row: the exact
build equals the FP64 oracle bit for bit at widths around the strips' edges,
with walls, potentials, self-gravity off and on, and at the largest grids that
take the kernels; the default tile gives the bits of the marching kernels
(which every other tile shape selects) on both sides of the rule."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

WALLS = [("reflect", "outflow"), ("periodic", "periodic"), ("reflect", "reflect")]
# 4096 waves of one and two strips, and one more row
EDGE = [(58, 64, 64), (59, 32, 64), (58, 64, 65), (59, 33, 63)]


def _problem(n, faces=None):
    p = W.blocks(3, n, seed=sum(n))
    if faces:
        p.bc = faces
    return p


def _grid(prob, prec, exact=True, **kw):
    from paper_1607_01105_amd.ppml import Grid

    print(f"[case] {prob.name} {prob.n} {prec} exact={exact} {kw}", flush=True)
    return Grid.from_problem(prob, prec=prec, exact=exact, **kw)


def _equal_oracle(g, o, steps):
    taus = o.run(steps)
    g.step(steps)
    t, dt, taken = g.time()
    assert taken == steps and t == o.t and dt == taus[-1]
    for f in range(6):
        assert np.array_equal(g.get(f), o.get(f)), f
    assert g.max_speeds() == o.max_speeds()


@pytest.mark.parametrize("faces", ["periodic", "walls", "outflow"])
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 3, 3), (7, 2, 5), (57, 6, 4), (58, 5, 7), (59, 9, 3), (116, 4, 6),
                               (117, 3, 8)] + EDGE[:2], ids=lambda n: "x".join(map(str, n)))
def test_exact_fp64_equals_oracle(n, faces):
    if faces == "walls" and (n[0] < 3 or n[2] < 3):
        pytest.skip("a reflecting axis needs three cells")
    prob = _problem(n, {"walls": WALLS, "outflow": [("outflow", "outflow")] * 3}.get(faces))
    _equal_oracle(_grid(prob, "fp64"), make_oracle(prob), 3)


@pytest.mark.parametrize("variant", ["first_order", "isothermal", "uniform", "log", "halo"])
def test_variants_equal_oracle(variant):
    prob = _problem((30, 20, 18), WALLS)
    kw = {}
    if variant == "first_order":
        kw["first_order"] = True
    elif variant == "isothermal":
        prob.isothermal = 0.8
        prob.p = 0.64 * prob.rho
    else:
        prob.potential = {"uniform": ("uniform", 0.3, -0.2, 0.1), "log": ("log", 0.5, 0.2, 0.9, 0.4, 0.5, 0.5),
                          "halo": ("halo", 0.3, 0.2, 0.6, 0.45, 0.5, 0.55)}[variant]
    g, o = _grid(prob, "fp64", **kw), make_oracle(prob, first_order=variant == "first_order")
    if variant != "halo":
        _equal_oracle(g, o, 4)
        return
    # the device's arctangent is not the oracle's: 1e-12 as for every FP64 product comparison
    o.run(4)
    g.step(4)
    for f in range(6):
        a, b = g.get(f), o.get(f)
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b)), f


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [(24, 31, 17), (61, 20, 12)] + EDGE, ids=lambda n: "x".join(map(str, n)))
def test_equals_marching_kernels(n, prec, exact):
    import torch

    prob = _problem(n, WALLS)
    a, b = _grid(prob, prec, exact), _grid(prob, prec, exact, tile=3)
    a.step(5)
    b.step(5)
    a.sync()
    b.sync()
    assert torch.equal(a.state, b.state) and a.time() == b.time() and a.max_speeds() == b.max_speeds()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_self_gravity_equals_marching_kernels(prec):
    import torch

    prob = W.gravity_sphere((30, 24, 20), seed=3, noise=0.05)
    a, b = _grid(prob, prec, False), _grid(prob, prec, False, tile=1)
    for g in (a, b):
        g.step(3)
        g.sync()
    assert torch.equal(a.state, b.state) and a.time() == b.time()
