"""The sine transforms at the block counts and launch shapes of ordinary runs:
FP32 transforms (every axis above 64 cells) at each count of 16-cell blocks, as
x, y and z axis; blocks of several waves, several groups of lines a block, and
FP64 tables that come in parts there.  Against a numpy solve for the same shell
values; bounds as for the potential (FP64 1e-12 normwise, FP32 5e-5)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1607_01105_amd import workloads as W
from test_gpu_sine_rounding import _solve

pytestmark = pytest.mark.gpu


def _check(n, prec):
    from paper_1607_01105_amd.ppml import Grid

    print(f"[case] {n} {prec}", flush=True)
    prob = W.gravity_sphere(n, L=1.0, noise=0.4, seed=sum(n), G=0.7)
    g = Grid.from_problem(prob, prec=prec)
    phi = g.potential()
    h = (prob.hi[0] - prob.lo[0]) / n[0]
    shell = phi.copy()
    shell[1:-1, 1:-1, 1:-1] = 0.0
    want = _solve(g.get(0), shell, 4.0 * np.pi * 0.7 * h * h)
    err = float(np.max(np.abs(phi[1:-1, 1:-1, 1:-1] - want)) / np.max(np.abs(want)))
    assert err <= (1e-12 if prec == "fp64" else 5e-5), (n, prec, err)


@pytest.mark.parametrize("m", [65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256])
def test_fp32_block_counts(m):
    for axis in range(3):
        n = [66, 70, 65]
        n[axis] = m
        _check(tuple(n), "fp32")


@pytest.mark.parametrize("n,prec", [((130, 130, 210), "fp64"), ((210, 182, 182), "fp64"), ((182, 210, 182), "fp64"),
                                    ((182, 182, 220), "fp32"), ((200, 130, 140), "fp32"), ((64, 182, 200), "fp32")],
                         ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_several_waves_and_groups(n, prec):
    _check(n, prec)
