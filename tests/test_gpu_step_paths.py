"""Single-launch steps of every deposit order: the resident launch and the
solve-first launches against tracer/solve launch pairs (timing mode), on
ragged sheets, open and closed, with and without per-segment charges."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I
from tests.parity import periodic_diff

pytestmark = pytest.mark.gpu

# sheets' tracer counts, cells, path
CASES = {
    # 9 chunks: a sheet of one tracer pair, partly filled and full chunks
    "resident_small": ([2, 65, 64, 130, 3, 63], 37, B.SIC_PATH_RESIDENT),
    # 32 chunks, four cells per solve thread
    "resident_full": ([512, 512, 400, 512], 1000, B.SIC_PATH_RESIDENT),
    # 33 chunks: the first size past the resident launch
    "step_small": ([64] * 33, 50, B.SIC_PATH_SOLVE_FIRST),
    "step_ragged": ([300, 77, 1000, 129, 64, 2, 641, 3000, 500], 256, B.SIC_PATH_SOLVE_FIRST),
    # 257 items: the first workgroup holds an item and writes the row
    "step_257_items": ([257] * 206 + [200, 3], 300, B.SIC_PATH_SOLVE_FIRST),
}


def _problem(counts, cells, charges):
    rng = np.random.default_rng(len(counts) + cells)
    L = 4.0 * np.pi
    nt = np.array(counts, dtype=np.int32)
    closed = np.array([0 if i % 3 == 1 else 1 for i in range(len(nt))], dtype=np.int32)
    x, v, c, q = [], [], [], []
    for i, n in enumerate(counts):
        s = np.arange(n) * (L / n)
        x.append(np.mod(s + 0.05 * np.sin(0.5 * s) + rng.uniform(0, L), L))
        v.append(np.full(n, -2.0 + 4.0 * i / max(1, len(counts) - 1)) + 0.01 * np.sin(s))
        q.append(L / len(counts) / (n if closed[i] else n - 1))
        c.append(q[-1] * (1.0 + 0.3 * np.sin(s)))
        if not closed[i]:
            c[-1][-1] = 0.0
    p = I.Problem(name="paths", L=L, n_cells=cells, dt=0.05, n_steps=0, n_tracers=nt, q=np.array(q), closed=closed)
    return p, np.concatenate(x), np.concatenate(v), np.concatenate(c) if charges else None


def _run(p, x, v, c, prec, order, calls, timing):
    with B.Simulation(p, precision=prec, x0=x, v0=v, deposit_order=order, seg_charges=c) as s:
        B.sic_set_timing(s.h, timing)
        paths = set()
        for n in calls:
            s.step(n)
            paths.add(B.sic_last_step_path(s.h))
        # one launch pair: it reads the halos and accumulators left behind
        B.sic_set_timing(s.h, True)
        s.step(1)
        return paths, s.state(), s.diagnostics()


@pytest.mark.parametrize("charges", [False, True])
@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("prec", [B.SIC_FP64, B.SIC_SPLIT_F32, B.SIC_SPLIT_U32])
@pytest.mark.parametrize("case", sorted(CASES))
def test_single_launch_steps_follow_the_launch_pairs(case, prec, order, charges):
    counts, cells, path = CASES[case]
    p, x, v, c = _problem(counts, cells, charges)
    print(f"case {case} prec={prec} order={order} charges={charges}", flush=True)
    calls = (1, 3, 45)  # the first step alone, direct launches, a graph and the steps left over
    paths, (xa, va, na), da = _run(p, x, v, c, prec, order, calls, False)
    _, (xb, vb, nb), db = _run(p, x, v, c, prec, order, (sum(calls),), True)
    assert paths == {path}
    assert na == nb == sum(calls) + 1
    ha, hb = da["history"], db["history"]
    assert np.array_equal(ha["step"], hb["step"]) and np.array_equal(ha["flags"], hb["flags"])
    if prec == B.SIC_FP64:
        # float64 atomics add in another order: rounding (1e-16 of the box a
        # step) grown over 50 steps, less than a period of the plasma
        assert np.max(periodic_diff(xa, xb, p.L)) < 1e-11 * p.L
        assert np.max(np.abs(va - vb)) < 1e-10
        np.testing.assert_allclose(ha["W_E"], hb["W_E"], rtol=1e-9)
    else:
        assert np.array_equal(xa, xb) and np.array_equal(va, vb)
        for col in ("W_E", "total_charge", "max_segment"):
            assert np.array_equal(ha[col], hb[col]), col
        assert np.array_equal(da["E"], db["E"]) and np.array_equal(da["rho"], db["rho"])
    # sums over the items in another order
    np.testing.assert_allclose(ha["KE"][:-1], hb["KE"][:-1], rtol=1e-11)
    scale = np.max(np.abs(hb["KE"][:-1])) * 2
    assert np.max(np.abs(ha["momentum"][:-1] - hb["momentum"][:-1])) < 1e-11 * scale


@pytest.mark.parametrize("order,cells,charges", [(0, 600, False), (0, 600, True), (1, 600, False), (2, 600, True),
                                                 (0, 3000, False), (1, 3000, False)])
@pytest.mark.parametrize("prec", [B.SIC_FP64, B.SIC_SPLIT_U32])
def test_long_runs_of_chunks_follow_the_work_items(prec, order, cells, charges):
    """A simulation of more than 512 work items steps with as many workgroups
    as run at a time; a tuned item size keeps the work items.  Several groups
    of 64 chunks per wavefront on 3000 cells, one on 600."""
    rng = np.random.default_rng(cells)
    m = 3000 if cells == 600 else 9000
    counts = rng.integers(600, 800, m)
    counts[:3] = (2, 64, 65)
    p, x, v, c = _problem([int(n) for n in counts], cells, charges)
    print(f"case runs prec={prec} order={order} cells={cells} charges={charges}", flush=True)
    res = []
    for tile in (0, 128):
        with B.Simulation(p, precision=prec, x0=x, v0=v, deposit_order=order, seg_charges=c, history_rows=16) as s:
            if tile:
                B.sic_set_tuning(s.h, tile_chunks=tile)
            else:
                assert B.sic_get_tuning(s.h)["grid_blocks"] > 512
            s.step(4)
            if not tile:
                assert B.sic_last_step_path(s.h) == B.SIC_PATH_FUSED
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
