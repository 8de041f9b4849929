"""What the host code launches, allocates and releases, on the CPU: libsic
bound to a runtime that records calls and runs nothing."""
import ctypes

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


def _sim(sheets=40, n=100, cells=64, order=0, **kw):
    p = I.landau(n_sheets=sheets, n_tracers=n, n_cells=cells, n_steps=1)
    return B.Simulation(p, precision=B.SIC_SPLIT_U32, deposit_order=order, stream=0, **kw)


@pytest.mark.parametrize("sheets,order", [(4, 0), (40, 0), (40, 1), (40, 2)])
@H.in_child
def test_a_first_step_call_prepares_nothing(sheets, order):
    # a caller may capture it: an allocation would fail, and what is only
    # recorded has not run when the next call starts
    with _sim(sheets=sheets, order=order) as s:
        H.rec.rec_clear()
        s.step(4)
        first = H.launches()
        assert "alloc" not in H.events()
        H.rec.rec_clear()
        s.step(4)
        assert H.launches() == first


@H.in_child
def test_a_failed_allocation_is_not_reported_again():
    H.rec.rec_fail_alloc(0)
    with pytest.raises(B.SicError):
        _sim()
    with _sim() as s:  # its launches are not blamed
        s.step(4)
        H.rec.rec_fail_alloc(0)
        with pytest.raises(B.SicError):
            s.set_state(0, s.problem.x0, s.problem.v0)
        s.step(4)


@pytest.mark.parametrize("at", range(13))
@H.in_child
def test_a_refining_call_that_finds_no_memory_leaves_nothing_half_done(at):
    with _sim(l_max=1.0, max_tracers=20000) as s:
        H.rec.rec_fail_alloc(at)  # one of the arrays of the first refining call
        with pytest.raises(B.SicError):
            s.step(3)
        H.rec.rec_fail_alloc(-1)
        s.step(3)  # and the next call has them all
        assert "null" not in H.events()
        assert H.rec.rec_live() > 0
    assert H.rec.rec_live() == 0


def _names(rows):
    return [next(n for n in ("k_step", "k_solve", "k_zero_mesh", "k_deposit", "k_refine_plan", "k_refine_rebuild")
                 if n in k) for k, *_ in rows]


@pytest.mark.parametrize("at", [0, 1, 4])
@H.in_child
def test_a_failed_launch_ends_the_run_at_the_steps_before_it(at):
    with _sim() as s:
        s.step(2)
        H.rec.rec_clear()
        H.rec.rec_fail_launch(b"k_step", at)
        with pytest.raises(B.SicError):
            s.step(6)
        # the solve that ends a run takes the charge of the last step that was launched
        assert _names(H.launches()) == ["k_step"] * at + ["k_solve"] * (at > 0)
        H.rec.rec_clear()
        s.step(2)
        assert _names(H.launches()) == ["k_step"] * 2 + ["k_solve"]


@H.in_child
def test_a_run_that_cannot_be_ended_starts_from_the_tracers_again():
    with _sim() as s:
        s.step(2)
        H.rec.rec_clear()
        H.rec.rec_fail_launch(b"k_solve", 0)
        with pytest.raises(B.SicError):
            s.step(3)
        assert _names(H.launches()) == ["k_step"] * 3 + ["k_zero_mesh"] * 3
        H.rec.rec_clear()
        s.step(2)
        assert _names(H.launches()) == ["k_deposit", "k_solve"] + ["k_step"] * 2 + ["k_solve"]


@H.in_child
def test_a_refining_run_that_cannot_be_ended_starts_from_the_tracers_again():
    with _sim(l_max=1.0, max_tracers=20000) as s:
        s.step(2)
        H.rec.rec_clear()
        H.rec.rec_fail_launch(b"k_refine_rebuild", 1)
        with pytest.raises(B.SicError):
            s.step(3)
        assert _names(H.launches()) == ["k_step", "k_refine_plan", "k_refine_rebuild", "k_deposit",
                                        "k_step", "k_refine_plan", "k_solve"] + ["k_zero_mesh"] * 3
        H.rec.rec_clear()
        s.step(1)
        assert _names(H.launches())[:3] == ["k_deposit", "k_solve", "k_step"]


@pytest.mark.parametrize("order", [0, 1])
@H.in_child
def test_a_launch_does_not_lower_the_lds_limit_of_larger_ones(order):
    # more than 512 work items: launches of as many workgroups as run at a time
    for cells in (4096, 3000, 2800):
        with _sim(sheets=1100, n=8192, cells=cells, order=order, history_rows=8) as s:
            s.step(2)
            assert "k_step" in H.launches()[-2][0]
    for cells in (4096, 2800, 2000, 300):
        with _sim(cells=cells, order=order) as s, _sim(sheets=4, cells=cells, order=order) as r:
            s.step(2)
            r.step(2)
            s.deposit()
    assert not [e for e in H.events() if e.startswith("lowered")]


@pytest.mark.parametrize("tuning", [{}, {"fused_only": 1}])
@H.in_child
def test_refining_calls_reuse_their_graphs_whichever_set_holds_the_state(tuning):
    with _sim(l_max=1.0, max_tracers=20000) as s:
        if tuning:
            B.sic_set_tuning(s.h, **tuning)
        for _ in range(2):  # both halo parities
            s.step(37)
        H.rec.rec_plan_inserts(1)
        s.step(37)  # one pass inserts: the other set holds the state
        H.rec.rec_plan_inserts(0)
        H.rec.rec_clear()
        for _ in range(2):
            s.step(37)
        assert "instantiate" not in H.events()


@H.in_child
def test_a_batch_solves_for_its_largest_live_mesh():
    def lds(b):
        H.rec.rec_clear()
        B.sic_batch_step(b, 2)
        return {row[3] for row in H.launches() if "k_solve" in row[0]}

    b = _batch(max_cells=4096)
    _admit(b, cells=64)
    assert lds(b) == {0}  # the solve of 16 cells per thread has its charge in LDS
    big = _admit(b, cells=1025)
    assert lds(b) == {2 * 8 * 17 * 256}
    B.sic_batch_release(b, big)
    assert lds(b) == {0}
    B.sic_batch_destroy(b)


@pytest.mark.parametrize("order,cells,chunks,size", [
    # twelve items per compute unit, from 48 chunks to 256
    (0, 1024, 20000, 48), (0, 1024, 150000, 56), (0, 1024, 900000, 256), (2, 256, 150000, 56),
    # four of piecewise-linear segments, up to 192 chunks
    (1, 1024, 20000, 48), (1, 1024, 150000, 168), (1, 1024, 900000, 192),
    # three quarters of one where the mesh leaves room for one workgroup
    (0, 4096, 10000, 64), (0, 4096, 20000, 120), (0, 4096, 150000, 256), (1, 3000, 10000, 64), (1, 3000, 150000, 192),
])
@H.in_child
def test_a_batch_sizes_its_items_by_arena_order_and_mesh(order, cells, chunks, size):
    b = B.sic_batch_create(chunks * 64, 1, cells, precision=B.SIC_SPLIT_U32, deposit_order=order, history_rows=8,
                           stream=0)
    _admit(b, cells=64, order=order)
    assert B.sic_batch_get_tuning(b)["tile_chunks"] == size
    B.sic_batch_destroy(b)


@H.in_child
def test_missing_device_outputs_are_refused_before_any_launch():
    with _sim() as s:
        H.rec.rec_clear()
        some = np.zeros(s.n).ctypes.data
        for x, v in ((None, None), (some, None), (None, some)):
            assert B.load().sic_get_state(s.h, x, v, None, B.SIC_MEM_DEVICE) == 1
        assert H.launches() == []
        assert B.load().sic_get_state(s.h, None, None, None, B.SIC_MEM_HOST) == 0


@H.in_child
def test_diagnostics_of_any_part_alone():
    lib, n = B.load(), ctypes.c_int64(0)
    rows = np.zeros(8, dtype=B.DIAG_DTYPE).ctypes.data
    mesh, last = np.zeros(64).ctypes.data, B.sic_diag()
    with _sim() as s:
        s.step(3)
        for args in ((None, None, None, None, ctypes.byref(n)), (ctypes.byref(last), None, None, None, None),
                     (None, mesh, None, None, None), (None, None, mesh, None, None),
                     (None, None, None, rows, ctypes.byref(n)), (None, None, None, None, None)):
            n.value = 8
            assert lib.sic_diagnostics(s.h, *args) == 0, args
    b = _batch()
    slot = _admit(b)
    assert lib.sic_batch_result(b, slot, None, None, None, None, ctypes.byref(n)) == 0
    B.sic_batch_result(b, slot, history=False)
    B.sic_batch_destroy(b)
