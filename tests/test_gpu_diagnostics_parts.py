"""Parts of a diagnostics call asked for alone."""
import ctypes

import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_length_and_newest_row_alone():
    p = I.landau(n_sheets=4, n_tracers=50, n_cells=33, alpha=0.05)
    with B.Simulation(p) as s:
        s.step(5)
        n = ctypes.c_int64(0)
        assert B.load().sic_diagnostics(s.h, None, None, None, None, ctypes.byref(n)) == 0 and n.value == 6
        d = B.sic_diagnostics(s.h, history=False)
        assert d["last"]["step"] == 5 and d["last"]["W_E"] == s.diagnostics()["last"]["W_E"]
