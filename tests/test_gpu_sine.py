"""The sine transforms of the self-gravity potential (Sec. 2.5), on the GPU
against the FP64 oracle, at the sizes where the kernels change: halves just
below, at and above a block of 16, one cell, tables that fill the LDS or come
in parts, the zero-padded block counts, and the first axis too long for the
kernels (library products) -- as x, y and z axis.

Bounds: those of the potential itself -- FP64 1e-12 (normwise, another order
of summation), FP32 5e-5 (rounding of the right-hand side and of three pairs
of length-N sums, amplified by the ratio of the eigenvalues).
"""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_oracle
from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 31, 32, 33, 63, 64, 65, 96, 97]
LONG = {"fp64": [160, 161, 192, 193, 256, 257], "fp32": [256, 257, 384, 385, 512, 513]}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_transform_sizes(prec, axis):
    from paper_1607_01105_amd.ppml import Grid

    for m in EDGES + LONG[prec]:
        n = [5, 6, 4]
        n[axis] = m
        prob = W.gravity_sphere(tuple(n), L=0.25 * n[0], noise=0.5, seed=m, G=0.8)
        print(f"[case] {n} {prec}", flush=True)
        ref = make_oracle(prob).potential()
        got = Grid.from_problem(prob, prec=prec).potential()
        err = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
        assert err <= (1e-12 if prec == "fp64" else 5e-5), (n, prec, err)
