"""Central differences of the closed forms, whose stencil points share their
centre's terms: dimensions around the wave's two rounds of 64 points and odd
ones, and smoothing probes as centres."""
import numpy as np
import pytest

import workloads as W
from test_gpu_closed_forms import FAMS, test_fd_gradient_matches_oracle_fd as check_fd
from test_gpu_phases import _gpu, _oracle_from, _rows_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", [n for n in FAMS if n != "bukin6"])
@pytest.mark.parametrize("d", [1, 2, 3, 16, 31, 32, 33, 63])
def test_fd_gradient_at_wave_edges(name, d):
    check_fd(name, d)


@pytest.mark.parametrize("name,d,M", [("rastrigin", 1, 20), ("michalewicz", 3, 5), ("michalewicz", 10, 4),
                                      ("styblinski_tang", 17, 3), ("ackley", 5, 10), ("trid", 4, 7)])
def test_smoothing_step_on_stencils_of_probes(name, d, M):
    """One smoothing step from a fixed state against the oracle; the tolerance
    is that of the mixtures' central-difference steps."""
    prob = W.closed_form_problem(name, d)
    cfg = W.RunConfig(N=120, m=5, n_osc=3, n_cloud=1, M=M, sigma=0.05, eps_grad=1e-3, grad_mode=0, seed=8)
    x0 = W.uniform_population(77, 120, prob.lo, prob.hi)
    with _gpu(prob, cfg, x0) as opt:
        opt.set_state(k=1)
        g0 = opt.get_state()
        opt.run_phases(1 << 5)
        g5 = opt.get_state()
    run = _oracle_from(prob, cfg, g0)
    run.phase_hlc()
    _rows_close(g5["X"].astype(np.float64) - g0["X"], run.X - g0["X"], 5e-3, "smoothing displacement", floor=1e-2)
