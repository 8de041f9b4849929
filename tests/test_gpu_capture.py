"""Steps captured by the caller and replayed: the state, the step that calls
report and the history follow the replays."""
import numpy as np
import pytest

from paper_1506_07207_amd import binding as B
from paper_1506_07207_amd import inputs as I

pytestmark = pytest.mark.gpu

# sheets, tracers, cells, path
CASES = {
    "resident": (4, 50, 33, B.SIC_PATH_RESIDENT),
    "solve_first": (40, 100, 64, B.SIC_PATH_SOLVE_FIRST),
}


def _equal(a, b, step):
    (xa, va, na), da = a.state(), a.diagnostics()
    (xb, vb, nb), db = b.state(), b.diagnostics()
    assert na == nb == step
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)
    assert np.array_equal(da["E"], db["E"]) and np.array_equal(da["rho"], db["rho"])
    assert list(da["history"]["step"]) == list(range(step + 1))
    for col in ("W_E", "total_charge", "max_segment", "flags"):
        assert np.array_equal(da["history"][col], db["history"][col]), col


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("order", [0, 1, 2])
def test_replayed_steps_are_reported(case, order):
    import torch

    sheets, tracers, cells, path = CASES[case]
    n = 4  # even: the halo buffers alternate, and a capture names them
    p = I.landau(n_sheets=sheets, n_tracers=tracers, n_cells=cells, alpha=0.05)
    print(f"case capture {case} order={order}", flush=True)
    stream = torch.cuda.Stream()
    with B.Simulation(p, precision=B.SIC_SPLIT_U32, deposit_order=order, stream=stream) as a, \
            B.Simulation(p, precision=B.SIC_SPLIT_U32, deposit_order=order) as b:
        a.step(n)
        b.step(n)
        assert B.sic_last_step_path(a.h) == path
        _equal(a, b, n)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
            a.step(n)
        _equal(a, b, n)  # captured, not run
        at = n
        for _ in range(3):
            with torch.cuda.stream(stream):
                graph.replay()
            b.step(n)
            at += n
            _equal(a, b, at)
            a.step(n)  # the simulation's own steps between
            b.step(n)
            at += n
            _equal(a, b, at)


@pytest.mark.parametrize("case", sorted(CASES))
def test_a_first_call_captured_and_dropped_changes_nothing(case):
    import torch

    sheets, tracers, cells, _ = CASES[case]
    p = I.landau(n_sheets=sheets, n_tracers=tracers, n_cells=cells, alpha=0.05)
    print(f"case capture dropped {case}", flush=True)
    stream = torch.cuda.Stream()
    with B.Simulation(p, precision=B.SIC_SPLIT_U32, stream=stream) as a, \
            B.Simulation(p, precision=B.SIC_SPLIT_U32) as b:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
            a.step(4)
        del graph
        _equal(a, b, 0)
        a.step(9)
        b.step(9)
        _equal(a, b, 9)
