"""Phase 1 with the active list kept in place (small classes) against the
compacted lists: a profiled handle takes the latter, and gives the same bits."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,kw", [(2, 1, {}), (3, 257, dict(grad_mode=0, ls_max=1)), (8, 3000, dict(ls_max=3)),
                                    (8, 16384, {}), (16, 100, dict(grad_mode=0)), (16, 4096, dict(ls_max=2)),
                                    (20, 2048, dict(m=3)), (64, 700, dict(noise=0.5))])
def test_same_bits_as_compacted_lists(d, N, kw):
    from paper_2606_26164_amd.api import Optimizer

    kw = dict(kw)
    prob = W.mixture_problem(700 + d, d, 5, 5.0, lam_range=(0.1, 1.0), noise_sigma=kw.pop("noise", 0.0))
    cfg = W.RunConfig(N=N, n_osc=4, n_conv=9, eps_grad=1e-3, seed=3, **kw)
    out = []
    for prof in (False, True):
        with Optimizer(prob, cfg, W.uniform_population(d, N, prob.lo, prob.hi)) as opt:
            if prof:
                opt.profile_begin()
            stats = opt.cycle(4, stats=True)
            st = opt.get_state(history=True)
        out.append((stats, st))
    assert out[0][0] == out[1][0]
    for f in ("X", "F", "G", "trace", "stuck", "active", "conv", "cnt", "head", "removed", "Wd"):
        assert np.array_equal(out[0][1][f], out[1][1][f], equal_nan=True), f


def test_closed_form_differences_in_place():
    from paper_2606_26164_amd.api import Optimizer

    prob = W.closed_form_problem("michalewicz", 7)
    cfg = W.RunConfig(N=300, n_osc=3, n_conv=8, eps_grad=1e-3, grad_mode=0, seed=4)
    out = []
    for prof in (False, True):
        with Optimizer(prob, cfg, W.uniform_population(1, 300, prob.lo, prob.hi)) as opt:
            if prof:
                opt.profile_begin()
            out.append((opt.cycle(3, stats=True), opt.get_state()["X"]))
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])
