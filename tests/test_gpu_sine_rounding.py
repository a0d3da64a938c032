"""FP32 self-gravity with an axis of at most 64 cells: the transforms run in FP64
between the stored density and the stored potential, so that the potential is
the exact solution for its own shell values, rounded once: within half a unit in
the last place (2^-24 of the value) and FP64's own error (1e-12 of the largest)
of a numpy solve."""
from __future__ import annotations

import numpy as np
import pytest

from paper_1607_01105_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solve(rho, shell, coef):
    """Interior potential: rho [z, y, x], the shell around zeros."""
    n = rho.shape
    b = coef * rho
    w = (0.0, 4.0 / 9.0, 1.0 / 9.0, 1.0 / 36.0)
    for dz in range(3):
        for dy in range(3):
            for dx in range(3):
                nd = (dz != 1) + (dy != 1) + (dx != 1)
                if nd:
                    b = b - w[nd] * shell[dz: dz + n[0], dy: dy + n[1], dx: dx + n[2]]
    f = []
    for m in n:
        j = np.arange(1, m + 1)
        f.append((np.sin(np.pi * ((j[:, None] * j) % (2 * m + 2)) / (m + 1)),
                  1.0 - 2.0 / 3.0 * np.sin(np.pi * j / (2.0 * (m + 1))) ** 2))

    def transform(a):
        for axis in range(3):
            a = np.moveaxis(np.tensordot(f[axis][0], a, (1, axis)), 0, axis)
        return a

    lam = -6.0 * (1.0 - f[0][1][:, None, None] * f[1][1][None, :, None] * f[2][1][None, None, :])
    return transform(transform(b) / lam) * np.prod([2.0 / (m + 1) for m in n])


@pytest.mark.parametrize("n", [(1, 2, 3), (2, 2, 2), (6, 6, 6), (17, 33, 16), (31, 65, 70), (64, 64, 64), (70, 65, 63),
                               (64, 100, 70), (130, 12, 97)], ids=lambda n: "x".join(map(str, n)))
def test_short_axes_round_once(n):
    from paper_1607_01105_amd.ppml import Grid

    for exact in (False, True):
        prob = W.gravity_sphere(n, L=1.0, noise=0.4, seed=sum(n), G=0.7)
        print(f"[case] {n} fp32 exact={exact}", flush=True)
        g = Grid.from_problem(prob, prec="fp32", exact=exact)
        phi = g.potential()
        h = (prob.hi[0] - prob.lo[0]) / n[0]
        shell = phi.copy()
        shell[1:-1, 1:-1, 1:-1] = 0.0
        want = _solve(g.get(0), shell, 4.0 * np.pi * 0.7 * h * h)
        err = np.abs(phi[1:-1, 1:-1, 1:-1] - want)
        assert np.all(err <= 2.0 ** -24 * np.abs(want) + 1e-12 * np.max(np.abs(want))), (n, err.max())
