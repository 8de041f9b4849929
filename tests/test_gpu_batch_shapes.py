"""Launch shapes of batches: what a batch stepped, or held, before a
simulation was admitted does not change that simulation's steps."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I

pytestmark = pytest.mark.gpu


def _admit(b, p, order, n_steps=-1):
    return B.sic_batch_admit(b, p.L, p.n_cells, p.dt, p.n_tracers, p.q, p.closed, p.x0, p.v0, n_steps,
                             precision=B.SIC_SPLIT_U32, deposit_order=order)


def _result(b, slot, p):
    x, v, step = B.sic_batch_get_state(b, slot, p.total_tracers)
    return x, v, step, B.sic_batch_result(b, slot, p.n_cells)


def _same(a, b):
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and a[2] == b[2]
    assert np.array_equal(a[3]["E"], b[3]["E"]) and np.array_equal(a[3]["rho"], b[3]["rho"])
    for col in ("step", "W_E", "total_charge", "max_segment", "flags"):
        assert np.array_equal(a[3]["history"][col], b[3]["history"][col]), col


@pytest.mark.parametrize("steps", [1, 2, 32])
@pytest.mark.parametrize("order", [0, 1, 2])
def test_steps_while_empty_do_not_change_what_is_admitted_later(order, steps):
    # 320 chunks, items of 48: against the tables of four chunks of an empty batch
    p = I.landau(n_sheets=40, n_tracers=500, n_cells=64)
    print(f"case empty batch order={order} steps={steps}", flush=True)
    out = []
    for empty_first in (False, True):
        b = B.sic_batch_create(40000, 4, 64, precision=B.SIC_SPLIT_U32, deposit_order=order)
        try:
            if empty_first:
                B.sic_batch_step(b, steps)
            slot = _admit(b, p, order)
            B.sic_batch_step(b, steps)
            out.append(_result(b, slot, p))
        finally:
            B.sic_batch_destroy(b)
    _same(*out)


@pytest.mark.parametrize("order", [0, 1, 2])
def test_larger_meshes_come_and_go(order):
    # the solve is built for the largest live mesh; every simulation's bits are
    # those it has alone in a batch
    sizes = [64, 256, 257, 1024, 1025, 3000]
    print(f"case batch meshes order={order}", flush=True)
    probs = [I.landau(n_sheets=4, n_tracers=300 + i, n_cells=c, alpha=0.05) for i, c in enumerate(sizes)]
    b = B.sic_batch_create(20000, 8, 4096, precision=B.SIC_SPLIT_U32, deposit_order=order)
    try:
        slots = []
        for p in probs:  # 5 steps with each further mesh
            slots.append(_admit(b, p, order))
            B.sic_batch_step(b, 5)
        first = _result(b, slots[0], probs[0])
        for k in range(len(probs) - 1, 0, -1):
            last = _result(b, slots[k], probs[k])
            alone = B.sic_batch_create(20000, 1, sizes[k], precision=B.SIC_SPLIT_U32, deposit_order=order)
            try:
                s = _admit(alone, probs[k], order)
                B.sic_batch_step(alone, last[2])
                _same(last, _result(alone, s, probs[k]))
            finally:
                B.sic_batch_destroy(alone)
            B.sic_batch_release(b, slots[k])
            B.sic_batch_step(b, 2)
        assert _result(b, slots[0], probs[0])[2] == first[2] + 2 * (len(probs) - 1)
        alone = B.sic_batch_create(20000, 1, sizes[0], precision=B.SIC_SPLIT_U32, deposit_order=order)
        try:
            s = _admit(alone, probs[0], order)
            B.sic_batch_step(alone, first[2] + 2 * (len(probs) - 1))
            _same(_result(b, slots[0], probs[0]), _result(alone, s, probs[0]))
        finally:
            B.sic_batch_destroy(alone)
    finally:
        B.sic_batch_destroy(b)
