"""Set and get calls move the caller's FP64 arrays in chunks of 1 MiB by several
threads: what is set is read back (FP64 bit for bit, FP32 rounded to nearest) at
sizes around the chunks' edges, from several Python threads at once, and every
refused value is refused wherever it lies, the state left as it was."""
from __future__ import annotations

import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(1,), (32768,), (131071,), (131072,), (131073,), (262144,), (262145,), (300, 437), (512, 513), (64, 64, 65),
         (96, 97, 98)]


def _grid(n, prec):
    from paper_1607_01105_amd.ppml import Grid

    return Grid(len(n), n, (0.0,) * len(n), (1.0,) * len(n), 1.4, 0.3, prec=prec)


def _fields(n, seed):
    rng = np.random.default_rng(seed)
    shp = tuple(n[::-1]) if len(n) == 3 else (1,) * (3 - len(n)) + tuple(n[::-1])
    e = rng.uniform(0.5, 2.0, shp)
    m = [rng.normal(0.0, 0.1, shp) if a < len(n) else None for a in range(3)]
    return [rng.uniform(0.5, 2.0, shp), *m, e + 5.0, e]


def _same(g, fields, prec):
    for f, a in enumerate(fields):
        if a is None:
            continue
        want = a if prec == "fp64" else a.astype(np.float32).astype(np.float64)
        assert np.array_equal(g.get(f), want), f


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_round_trip(n, prec):
    g = _grid(n, prec)
    fields = _fields(n, sum(n))
    g.set_conserved(fields, rho_mean0=1.0, t=0.25)
    _same(g, fields, prec)
    tot = g.totals()
    for f, a in enumerate(fields):
        if a is not None:
            # 2-pass FP64 sums in another order, of values rounded to the storage type
            want = a if prec == "fp64" else a.astype(np.float32).astype(np.float64)
            assert abs(tot[f] - want.sum()) <= 1e-12 * np.abs(want).sum()
    fields[1] = None  # an absent momentum is zero
    g.set_conserved(fields, rho_mean0=1.0, t=0.25)
    assert not g.get(1).any()


def test_refused_values_leave_the_state():
    from paper_1607_01105_amd.ppml import PPMLError

    n = (300, 437)
    g = _grid(n, "fp64")
    good = _fields(n, 3)
    g.set_conserved(good, rho_mean0=1.0)
    N = n[0] * n[1]
    for f, bad in ((0, 0.0), (0, np.nan), (0, np.inf), (1, np.nan), (2, -np.inf), (4, np.nan), (5, -1.0), (5, np.inf)):
        for at in (0, N // 2, N - 1):
            fields = [None if a is None else a.copy() for a in good]
            fields[f].reshape(-1)[at] = bad
            with pytest.raises(PPMLError):
                g.set_conserved(fields, rho_mean0=1.0)
            rho, u, v, _, _, p = fields
            if f in (0, 1, 2, 5):
                with pytest.raises(PPMLError):
                    g.set_primitive(rho, u, v, None, p)
    _same(g, good, "fp64")


def test_threads_at_once():
    grids = [(_grid((200, 300 + 17 * i), p), _fields((200, 300 + 17 * i), i), p) for i, p in enumerate(["fp32", "fp64"] * 3)]
    failed = []

    def work(g, fields, prec):
        try:
            for _ in range(5):
                g.set_conserved(fields, rho_mean0=1.0)
                _same(g, fields, prec)
        except BaseException as e:  # noqa: BLE001 -- reported by the main thread
            failed.append(e)

    ts = [threading.Thread(target=work, args=a) for a in grids]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not failed, failed[0]
