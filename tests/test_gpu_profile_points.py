"""A profile of a small problem times the launches that its runs make and counts
the points that they compute."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _profile(d, N, **kw):
    from paper_2606_26164_amd.api import Optimizer

    prob = W.mixture_problem(31, d, 6, 6.0, lam_range=(0.1, 1.0))
    cfg = W.RunConfig(N=N, n_osc=3, n_conv=9, M=4, eps_grad=1e-3, seed=3, **kw)
    with Optimizer(prob, cfg, W.uniform_population(d, N, prob.lo, prob.hi)) as opt:
        opt.profile_begin()
        stats = opt.cycle(2, stats=True)
        return opt.profile_end(), sum(s["evals"] for s in stats)


EVALS = ("eval_direct", "eval_trial", "eval_probe", "eval_fd")


# in place (the first four of them), with lists, with the trials in stages
@pytest.mark.parametrize("d,N,kw", [(3, 300, {}), (8, 9000, dict(grad_mode=0)), (16, 1500, {}), (30, 700, {}),
                                    (16, 4000, {}), (40, 9000, {})])
def test_every_direction_is_followed_by_one_first_trial(d, N, kw):
    prof, evals = _profile(d, N, ls_max=1, **kw)
    assert prof["lbfgs"]["points"] == prof["eval_trial"]["points"] > N
    assert prof["lbfgs_pairs"]["points"] > 0
    # one trial a search: nothing is computed that a stage would not need
    assert sum(prof[k]["points"] for k in EVALS if k in prof) == evals


@pytest.mark.parametrize("d,N,merged", [(3, 300, True), (16, 4000, True), (40, 9000, False)])
def test_points_are_those_computed(d, N, merged):
    """Merged launches compute all trials of a search that rejects t = 1."""
    prof, evals = _profile(d, N, ls_max=10)
    points = sum(prof[k]["points"] for k in EVALS if k in prof)
    assert points > evals if merged else points == evals
