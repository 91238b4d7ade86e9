"""A closed form's central differences take no schedule: nothing is to be
chosen from the scatter of four timings of one launch."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,d,N", [("michalewicz", 64, 4000), ("rastrigin", 5, 60000), ("bukin6", 2, 500)])
def test_closed_form_difference_class_keeps_the_default(name, d, N):
    from paper_2606_26164_amd.api import Optimizer

    prob = W.closed_form_problem(name, d)
    cfg = W.RunConfig(N=N, n_osc=2, eps_grad=1e-3, grad_mode=0, seed=4)
    for _ in range(3):
        with Optimizer(prob, cfg, W.uniform_population(1, N, prob.lo, prob.hi)) as opt:
            (t,) = opt.tuning()
        assert len(set(t["ms"])) == 1 and t["ms"][0] > 0
        assert (t["order"], t["grid_cap"]) == (0, 8192)
