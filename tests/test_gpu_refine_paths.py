"""Refining steps on the device, solve-first or as launch pairs, against the
host's passes (timing mode) on ragged sheets, open and closed: the same
tracers in the same order, the same field."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I
from tests.parity import periodic_diff

pytestmark = pytest.mark.gpu

COUNTS = [2, 63, 64, 65, 128, 3, 127, 200, 1, 500]


def _problem(cells):
    rng = np.random.default_rng(cells)
    L = 4.0 * np.pi
    counts = [max(2, n) for n in COUNTS]
    closed = np.array([0 if i % 3 == 1 else 1 for i in range(len(counts))], dtype=np.int32)
    x, v, q = [], [], []
    for i, n in enumerate(counts):
        s = np.arange(n) * (L / n)
        x.append(np.mod(s + 0.2 * np.sin(0.5 * s) + rng.uniform(0, L), L))
        v.append(20.0 * np.sin(2.0 * s + i))  # sheared: segments stretch by up to 40 times
        q.append(L / len(counts) / (n if closed[i] else n - 1))
    p = I.Problem(name="refine", L=L, n_cells=cells, dt=0.02, n_steps=0,
                  n_tracers=np.array(counts, dtype=np.int32), q=np.array(q), closed=closed)
    return p, np.concatenate(x), np.concatenate(v)


def _run(p, x, v, prec, order, calls, l_max, capacity, timing=False, **tuning):
    with B.Simulation(p, precision=prec, x0=x, v0=v, deposit_order=order, l_max=l_max, max_tracers=capacity) as s:
        if tuning:
            B.sic_set_tuning(s.h, **tuning)
        B.sic_set_timing(s.h, timing)
        for n in calls:
            s.step(n)
        out = s.layout()[0], s.state(), s.charges(), s.diagnostics()
        # a further call on the host's passes: it takes over the layout, the
        # halos, the charge edges and the accumulators
        B.sic_set_timing(s.h, True)
        s.step(1)
        return out, (s.layout()[0], s.state(), s.charges(), s.diagnostics())


@pytest.mark.parametrize("tuning", [{}, {"fused_only": 1}, {"tile_chunks": 4, "block_threads": 256}])
@pytest.mark.parametrize("order", [0, 1, 2])
@pytest.mark.parametrize("prec", [B.SIC_FP64, B.SIC_SPLIT_F32, B.SIC_SPLIT_U32])
def test_device_passes_follow_the_host_passes(prec, order, tuning):
    p, x, v = _problem(48)
    print(f"case refine paths prec={prec} order={order} {tuning}", flush=True)
    l_max, capacity = 1.5 * p.L / p.n_cells, 40000
    calls = (1, 2, 8, 40)  # a step alone, direct launches, a graph, two graphs
    got = _run(p, x, v, prec, order, calls, l_max, capacity, **tuning)
    want = _run(p, x, v, prec, order, (sum(calls),), l_max, capacity, timing=True)
    assert int(want[0][0].sum()) > 3 * int(p.n_tracers.sum())  # many passes inserted
    for a, b in zip(got, want):
        assert np.array_equal(a[0], b[0])
        assert a[1][2] == b[1][2]
        ha, hb = a[3]["history"], b[3]["history"]
        assert np.array_equal(ha["step"], hb["step"]) and np.array_equal(ha["flags"], hb["flags"])
        assert np.array_equal(a[2], b[2])  # halves are exact in every form
        if prec == B.SIC_FP64:
            # float64 sums in another order, over 52 steps of dt 0.02
            assert np.max(periodic_diff(a[1][0], b[1][0], p.L)) < 1e-11 * p.L
            np.testing.assert_allclose(ha["W_E"], hb["W_E"], rtol=1e-9)
            np.testing.assert_allclose(ha["max_segment"], hb["max_segment"], rtol=1e-9)
        else:
            assert np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])
            assert np.array_equal(ha["W_E"], hb["W_E"]) and np.array_equal(ha["max_segment"], hb["max_segment"])
        np.testing.assert_allclose(ha["KE"][:-1], hb["KE"][:-1], rtol=1e-9)


@pytest.mark.parametrize("fused_only", [0, 1])
def test_refused_pass_leaves_the_simulation_at_its_step(fused_only):
    p, x, v = _problem(48)
    l_max = 1.5 * p.L / p.n_cells
    with B.Simulation(p, precision=B.SIC_SPLIT_U32, x0=x, v0=v, l_max=l_max, max_tracers=3000) as s:
        B.sic_set_tuning(s.h, fused_only=fused_only)
        with pytest.raises(B.SicError):
            s.step(60)
        nt, (xs, vs, at), d = s.layout()[0], s.state(), s.diagnostics()
        assert 0 < at < 60 and int(nt.sum()) <= 3000
        assert d["last"]["step"] == at == len(d["history"]) - 1
    # the same run with room, up to the step before and through the refused one
    with B.Simulation(p, precision=B.SIC_SPLIT_U32, x0=x, v0=v, l_max=l_max, max_tracers=40000) as s:
        s.step(at - 1)
        assert np.array_equal(s.layout()[0], nt)
        s.step(1)
        assert int(s.layout()[0].sum()) > 3000
