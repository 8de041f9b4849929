"""Solve-first steps whose first workgroup holds a work item and writes the
row after it (256 workgroups: one per compute unit), and the largest resident
simulation: every deposit order, with and without per-segment charges, against
tracer/solve launch pairs."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from tests import host_runtime as H
from tests.parity import periodic_diff
from tests.test_gpu_step_paths import _problem, _run

# sheets' tracer counts, cells, path, step launch's workgroups and threads
CASES = {
    # 1023 chunks: 256 items of 4, the last of 3
    "items_256": ([257] * 204 + [190], 300, B.SIC_PATH_SOLVE_FIRST, 256, 256),
    # 8170 and 8192 chunks: 511 and 512 items of 16, taken two at a time
    "items_511": ([640] * 816 + [639], 256, B.SIC_PATH_SOLVE_FIRST, 256, 1024),
    "items_512": ([640] * 819 + [65], 256, B.SIC_PATH_SOLVE_FIRST, 256, 1024),
    # 32 chunks: the last size that is resident, four cells per solve thread
    "resident_32": ([512, 512, 460, 512], 1000, B.SIC_PATH_RESIDENT, 1, 13 * 64),
}


@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("case", sorted(CASES))
@H.in_child
def test_the_cases_take_these_launches(case, order):
    counts, cells, path, grid, block = CASES[case]
    p, x, v, _ = _problem(counts, cells, False)
    with B.Simulation(p, precision=B.SIC_SPLIT_U32, x0=x, v0=v, deposit_order=order, stream=0) as s:
        H.rec.rec_clear()
        s.step(1)
        assert B.sic_last_step_path(s.h) == path
        kernel, *shape = H.launches()[0][:3]
        assert ("k_resident" if path == B.SIC_PATH_RESIDENT else "k_step") in kernel
        assert shape == [grid, block]


@pytest.mark.gpu
@pytest.mark.parametrize("charges", [False, True])
@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("prec", [B.SIC_FP64, B.SIC_SPLIT_U32])
@pytest.mark.parametrize("case", sorted(CASES))
def test_the_row_after_the_item_follows_the_launch_pairs(case, prec, order, charges):
    counts, cells, path, _, _ = CASES[case]
    p, x, v, c = _problem(counts, cells, charges)
    print(f"case {case} prec={prec} order={order} charges={charges}", flush=True)
    calls = (1, 2, 20)  # the first step alone, direct launches, a graph
    paths, (xa, va, na), da = _run(p, x, v, c, prec, order, calls, False)
    _, (xb, vb, nb), db = _run(p, x, v, c, prec, order, (sum(calls),), True)
    assert paths == {path}
    assert na == nb == sum(calls) + 1
    ha, hb = da["history"], db["history"]
    assert np.array_equal(ha["step"], hb["step"]) and np.array_equal(ha["flags"], hb["flags"])
    if prec == B.SIC_FP64:
        # float64 sums in another order: rounding (1e-16 of the box a step)
        # grown over 23 steps of 0.05, a fifth of a plasma period
        assert np.max(periodic_diff(xa, xb, p.L)) < 1e-11 * p.L
        assert np.max(np.abs(va - vb)) < 1e-10
        for col in ("W_E", "total_charge", "max_segment"):
            np.testing.assert_allclose(ha[col], hb[col], rtol=1e-9)
    else:
        assert np.array_equal(xa, xb) and np.array_equal(va, vb)
        for col in ("W_E", "total_charge", "max_segment"):
            assert np.array_equal(ha[col], hb[col]), col
        assert np.array_equal(da["E"], db["E"]) and np.array_equal(da["rho"], db["rho"])
    # sums over the items in another order
    np.testing.assert_allclose(ha["KE"][:-1], hb["KE"][:-1], rtol=1e-11)
    scale = np.max(np.abs(hb["KE"][:-1])) * 2
    assert np.max(np.abs(ha["momentum"][:-1] - hb["momentum"][:-1])) < 1e-11 * scale
