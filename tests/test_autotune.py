"""The tile-shape tuner: a shape other than the default has to win by more than
the timings' noise, and what is timed is what runs."""
from __future__ import annotations

import pytest

from paper_1607_01105_amd import workloads as W


def test_choose_needs_a_gain_beyond_the_noise():
    from paper_1607_01105_amd.autotune import choose

    assert choose({0: [1.0, 1.0, 1.2], 1: [0.5, 0.6, 0.5]}) == (1, {0: 1.0, 1: 0.5})
    assert choose({0: [1.0, 1.0, 1.0], 1: [0.99, 0.99, 0.99]})[0] == 0   # within the margin
    assert choose({0: [1.0, 1.2, 1.3], 1: [0.9, 0.9, 0.9]})[0] == 0      # within the default's own spread
    assert choose({0: [1.3, 1.0, 1.01], 1: [0.9, 0.9, 0.9]})[0] == 1     # a cold first call is no spread
    assert choose({0: [1.0, 1.0, 1.0]}) == (0, {0: 1.0})


@pytest.mark.gpu
def test_short_lines_and_sheets(monkeypatch):
    """1-D grids that take the line kernel are timed through it (a third of the
    stage kernels' time at 512 cells FP64; half is asked), and neither they nor
    2-D grids, whose kernels have no tiles, get a shape of their own."""
    import torch

    from paper_1607_01105_amd import autotune
    from paper_1607_01105_amd.ppml import Grid

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("PPML_AUTOTUNE_CACHE", "")
    line = W.blocks(1, (512,), seed=11)
    print("[case] tune_grid 1-D 512 fp64", flush=True)
    r = autotune.tune_grid(line, prec="fp64", steps=64, warmup=64)
    assert r["tile"] == 0 and set(r["ms_per_step"]) == {0, 1, 2}
    g = Grid.from_problem(line, prec="fp64")
    g.set_timing(64)
    g.step(64)
    a, b, n = g.get_timing()
    assert n == 64 and r["ms_per_step"][0] < 0.5 * (a + b) / n
    for prob in (W.blocks(2, (64, 48), seed=12), W.blocks(2, (200, 300), seed=13)):
        print(f"[case] tune_grid {prob.name} fp32", flush=True)
        assert autotune.tune_grid(prob, prec="fp32")["tile"] == 0
