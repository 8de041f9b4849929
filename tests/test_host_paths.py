"""What the host code launches, allocates and releases, on the CPU: libsic
bound to a runtime that records calls and runs nothing."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I
from tests import host_runtime as H


def _batch(max_cells=64, budget=40000, slots=4, order=0, flags=0):
    return B.sic_batch_create(budget, slots, max_cells, precision=B.SIC_SPLIT_U32, deposit_order=order, flags=flags,
                              stream=0)


def _admit(b, cells=64, sheets=8, n=500, order=0, n_steps=-1, **kw):
    p = I.landau(n_sheets=sheets, n_tracers=n, n_cells=cells, n_steps=1)
    return B.sic_batch_admit(b, p.L, p.n_cells, p.dt, p.n_tracers, p.q, p.closed, p.x0, p.v0, n_steps,
                             precision=B.SIC_SPLIT_U32, deposit_order=order, **kw)


@pytest.mark.parametrize("steps", [2, 32])
@pytest.mark.parametrize("order", [0, 1, 2])
@H.in_child
def test_steps_of_an_empty_batch_leave_no_launch_for_the_simulations_admitted_later(steps, order):
    def run(empty_first):
        b = _batch(order=order)
        if empty_first:
            B.sic_batch_step(b, steps)
        _admit(b, order=order)
        H.rec.rec_clear()
        B.sic_batch_step(b, steps)
        got = H.launches()
        B.sic_batch_destroy(b)
        return got

    assert run(True) == run(False)
