"""2-D grids, whose stage kernels give a wave a strip of up to 58 columns and a
few rows: the exact build equals the FP64 oracle bit for bit at widths and
heights around the strips' edges and for every face kind; a grid's bits do not
depend on the rows per wave that its launch takes, alone or in batches of
other sizes; in a batch, long 1-D grids that step beside 2-D grids keep the
bits of the stage kernels."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

FACES = {"periodic": None, "outflow": [("outflow", "outflow")] * 2, "walls": [("reflect", "outflow"), ("reflect", "reflect")],
         "inflow": [("inflow", "outflow"), ("reflect", "inflow")]}


def _problem(n, faces="periodic"):
    p = W.blocks(2, n, seed=n[0] + n[1])
    if FACES[faces]:
        p.bc = FACES[faces] + p.bc[2:]
    if faces == "inflow":
        p.inflow = {0: (1.4, 0.7, 0.2, 0.0, 1.0), 3: (0.8, -0.1, -0.5, 0.0, 0.7)}
    return p


def _grid(prob, prec, exact=True):
    from paper_1607_01105_amd.ppml import Grid

    print(f"[case] {prob.name} {prob.n[:2]} {prec} exact={exact}", flush=True)
    return Grid.from_problem(prob, prec=prec, exact=exact)


# one and several rows per wave (the last three), narrow and ragged strips
SIZES = [(1, 1), (2, 5), (8, 3), (57, 4), (58, 5), (59, 6), (64, 64), (66, 33), (116, 7), (117, 8), (175, 61), (300, 401),
         (464, 257)]


@pytest.mark.parametrize("faces", list(FACES))
@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_exact_fp64_equals_oracle(n, faces):
    if min(n) < 3 and faces in ("walls", "inflow"):
        pytest.skip("a reflecting axis needs three cells")
    prob = _problem(n, faces)
    o = make_oracle(prob)
    taus = o.run(4)
    g = _grid(prob, "fp64")
    g.step(4)
    t, dt, taken = g.time()
    assert taken == 4 and t == o.t and dt == taus[-1]
    for f in (0, 1, 2, 4, 5):
        assert np.array_equal(g.get(f), o.get(f)), f
    assert g.max_speeds() == o.max_speeds()


# the second grid sets the rows per wave of the launch: FP32 2, 3, 4, 8; FP64 2
@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("prec,big", [("fp32", (256, 300)), ("fp32", (371, 371)), ("fp32", (512, 700)),
                                      ("fp32", (1400, 1500)), ("fp64", (300, 401))])
def test_rows_per_wave_do_not_change_bits(prec, big, exact):
    import torch

    from paper_1607_01105_amd.ppml import Batch

    small = [_problem((70, 45), "walls"), _problem((33, 66), "inflow"), _problem((5, 3))]
    probs = small + [_problem(big, "outflow")]
    b = Batch(capacity=len(probs), exact=exact)
    slots = [b.admit(b.new_grid(p, prec=prec)) for p in probs]
    b.step(5)
    b.sync()
    for p, s in zip(probs, slots):
        solo = _grid(p, prec, exact)
        solo.step(5)
        solo.sync()
        assert torch.equal(solo.state, b.grids[s].state), p.n
        assert solo.time() == b.grids[s].time()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_long_line_grids_beside_2d_grids(prec):
    import torch

    from paper_1607_01105_amd.ppml import Batch

    probs = [W.blocks(1, (n,), seed=n, bc=bc) for n, bc in ((4608, "outflow"), (4609, "periodic"), (3900, "periodic"),
                                                            (2305, "reflect"), (100, "outflow"))]
    probs.append(_problem((40, 30)))
    for steps in (6, 7):  # the last step's buffer: the stage output and the state
        b = Batch(capacity=8, exact=True)
        slots = [b.admit(b.new_grid(p, prec=prec)) for p in probs]
        b.step(steps)
        b.sync()
        for p, s in zip(probs, slots):
            solo = _grid(p, prec)
            solo.step(steps)
            solo.sync()
            assert torch.equal(solo.state, b.grids[s].state), p.n
            assert solo.time() == b.grids[s].time() and solo.max_speeds() == b.grids[s].max_speeds()
