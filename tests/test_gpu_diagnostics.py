"""Diagnostics calls: one block of host memory per call up to 1024 history
rows, copies above; the ring's wrap; the step that calls report."""
import ctypes

import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I

pytestmark = pytest.mark.gpu


def _newest(s, n):
    """The newest n rows through the C entry point."""
    rows = np.zeros(n, dtype=B.DIAG_DTYPE)
    got = ctypes.c_int64(n)
    assert B.load().sic_diagnostics(s.h, None, None, None, rows.ctypes.data_as(ctypes.c_void_p), ctypes.byref(got)) == 0
    return rows[: got.value]


@pytest.mark.parametrize("steps", [0, 1, 1022, 1023, 1024, 1500])
def test_history_across_the_block_and_the_copies(steps):
    # 1023 steps: 1024 rows, the most that the block holds; compared with the
    # same run (bitwise reproducible in the split form) read 100 steps at a time
    p = I.landau(n_sheets=4, n_tracers=50, n_cells=33, alpha=0.05)
    with B.Simulation(p, precision=B.SIC_SPLIT_U32) as a, B.Simulation(p, precision=B.SIC_SPLIT_U32) as b:
        a.step(steps)
        d = a.diagnostics()
        parts = [b.diagnostics()["history"][:1]]
        for at in range(0, steps, 100):
            n = min(100, steps - at)
            b.step(n)
            parts[-1] = parts[-1][:-1]  # the newest row's kinetic energy waits for the next move
            parts.append(_newest(b, n + 1))
        want = np.concatenate(parts)
        assert a.state()[2] == steps
        assert list(d["history"]["step"]) == list(range(steps + 1))
        for col in B.DIAG_DTYPE.names:
            assert np.array_equal(d["history"][col], want[col], equal_nan=True), col
            assert np.array_equal(d["last"][col], want[col][-1], equal_nan=True), col
        e = b.diagnostics()
        assert np.array_equal(d["E"], e["E"]) and np.array_equal(d["rho"], e["rho"])


@pytest.mark.parametrize("rows,steps", [(16, 15), (16, 16), (16, 40), (1200, 2500)])
def test_history_ring_wraps(rows, steps):
    p = I.landau(n_sheets=4, n_tracers=50, n_cells=33, alpha=0.05)
    with B.Simulation(p, precision=B.SIC_SPLIT_U32, history_rows=rows) as a, \
            B.Simulation(p, precision=B.SIC_SPLIT_U32) as b:
        a.step(steps)
        b.step(steps)
        h, full = a.diagnostics()["history"], b.diagnostics()["history"]
        n = min(rows, steps + 1)
        assert list(h["step"]) == list(range(steps + 1 - n, steps + 1))
        for col in B.DIAG_DTYPE.names:
            assert np.array_equal(h[col], full[col][-n:], equal_nan=True), col


def test_step_reported_by_every_way_of_stepping():
    p = I.landau(n_sheets=4, n_tracers=50, n_cells=33, alpha=0.05)
    with B.Simulation(p, precision=B.SIC_SPLIT_U32) as s:
        def step():
            d = s.diagnostics()
            assert d["last"]["step"] == d["history"]["step"][-1] == s.state()[2]
            return d["last"]["step"]

        assert step() == 0
        for k in (1, 2):  # by hand
            s.push()
            s.deposit()
            s.solve()
            assert step() == k
        s.deposit()
        s.solve()  # no move: the same step
        assert step() == 2
        s.step(7)
        assert step() == 9
        B.sic_set_timing(s.h, True)
        s.step(3)
        assert step() == 12
        x, v, _ = s.state()
        s.set_state(100, x, v)
        s.step(0)
        assert step() == 100 and len(s.diagnostics()["history"]) == 1
        B.sic_autotune(s.h, 1)
        assert step() == 100
        s.load_state(7, p.n_tracers, x, v)
        s.step(1)
        assert step() == 8
