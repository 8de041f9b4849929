"""Steps of a single simulation of more than 512 work items: one workgroup per
item, or as many workgroups as run at a time through all chunks together."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from tests import host_runtime as H
from tests.parity import periodic_diff
from tests.test_gpu_step_paths import _problem

# order, precision, per-segment charges, cells; whether 8.4M tracers step in runs
CHOICES = [
    (0, B.SIC_FP64, False, 1024, True), (0, B.SIC_SPLIT_U32, True, 1024, True),
    (2, B.SIC_FP64, False, 1024, True), (2, B.SIC_SPLIT_U32, False, 1024, False),
    (1, B.SIC_FP64, False, 1024, False), (1, B.SIC_SPLIT_F32, True, 1024, False),
    (1, B.SIC_SPLIT_U32, True, 1200, True), (1, B.SIC_SPLIT_U32, False, 1200, False),
    (2, B.SIC_SPLIT_F32, False, 1200, True), (1, B.SIC_FP64, False, 3000, True),
]


@pytest.mark.parametrize("order,prec,charges,cells,runs", CHOICES)
@H.in_child
def test_runs_are_taken_where_they_pay(order, prec, charges, cells, runs):
    n = 8 << 20
    x, v = np.linspace(0.0, 12.0, n, endpoint=False), np.zeros(n)
    c = np.full(n, 1.0 / n) if charges else None
    h = B.sic_init(12.0, cells, 0.05, [n], [1.0 / n], [1], x, v, precision=prec, deposit_order=order, seg_charges=c,
                   history_rows=8, stream=0)
    assert B.sic_get_tuning(h)["grid_blocks"] > 512
    H.rec.rec_clear()
    B.sic_step(h, 1)
    kernel = H.launches()[0][0]
    assert ("k_step" if runs else "k_tracers") in kernel, kernel
    B.sic_destroy(h)


@pytest.mark.parametrize("items,charges,per_cu,grid", [
    (600, False, 1, 200), (600, False, 2, 600), (600, False, 3, 600), (600, True, 2, 600),
    (820, False, 2, 410), (820, True, 2, 820), (1024, False, 2, 512), (1024, True, 2, 512), (1024, False, 1, 256),
])
@H.in_child
def test_deposits_run_where_the_runs_fill_the_machine(items, charges, per_cu, grid):
    n = items * 128 * 64  # 2048 cells: items of 128 chunks
    x, v = np.linspace(0.0, 12.0, n, endpoint=False), np.zeros(n)
    c = np.full(n, 1.0 / n) if charges else None
    h = B.sic_init(12.0, 2048, 0.05, [n], [1.0 / n], [1], x, v, seg_charges=c, history_rows=8, stream=0)
    assert B.sic_get_tuning(h)["grid_blocks"] == items
    H.rec.rec_clear()
    H.rec.rec_occupancy(per_cu)
    B.sic_deposit(h)
    assert H.launches()[-1][1] == grid
    B.sic_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("order,charges", [(0, True), (1, False), (1, True), (2, False), (2, True)])
@pytest.mark.parametrize("prec", [B.SIC_FP64, B.SIC_SPLIT_F32, B.SIC_SPLIT_U32])
def test_runs_follow_the_work_items(prec, order, charges):
    # 70 000 chunks on 1200 cells, items of 76 chunks: runs in every form; a
    # tuned item size keeps the work items
    rng = np.random.default_rng(order)
    counts = rng.integers(3800, 4300, 1100)
    counts[:3] = (2, 64, 65)
    p, x, v, c = _problem([int(n) for n in counts], 1200, charges)
    print(f"case runs prec={prec} order={order} charges={charges}", flush=True)
    res = []
    for tile in (0, 128):
        with B.Simulation(p, precision=prec, x0=x, v0=v, deposit_order=order, seg_charges=c, history_rows=16) as s:
            if tile:
                B.sic_set_tuning(s.h, tile_chunks=tile)
            s.step(4)
            res.append((s.state(), s.diagnostics()))
    (xa, va, na), da = res[0]
    (xb, vb, nb), db = res[1]
    assert na == nb == 4
    if prec == B.SIC_FP64:
        # float64 sums of up to 1e5 additions per cell in another order
        assert np.max(periodic_diff(xa, xb, p.L)) < 1e-12 * p.L
        np.testing.assert_allclose(da["history"]["W_E"], db["history"]["W_E"], rtol=1e-9)
    else:
        assert np.array_equal(xa, xb) and np.array_equal(va, vb)
        assert np.array_equal(da["E"], db["E"])
        assert np.array_equal(da["history"]["max_segment"], db["history"]["max_segment"])
    np.testing.assert_allclose(da["history"]["KE"][:-1], db["history"]["KE"][:-1], rtol=1e-11)
