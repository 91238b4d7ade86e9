"""Phase 1 with the active list kept in place against compacted lists: a problem
alone (its class small) and beside one that makes the class large."""
import pytest

import workloads as W
from test_gpu_batch import _assert_same, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,big,kw", [(2, 1, 17000, {}), (3, 257, 17000, dict(grad_mode=0, ls_max=1)),
                                        (8, 3000, 16000, dict(ls_max=3)), (16, 100, 2100, dict(grad_mode=0)),
                                        (16, 2000, 2100, dict(ls_max=2)), (20, 900, 1100, dict(m=3)),
                                        (32, 700, 1100, dict(noise=0.5)), (5, 800, 17000, dict(noise=0.3, grad_mode=0))])
def test_same_bits_as_compacted_lists(d, N, big, kw):
    from paper_2606_26164_amd.api import Optimizer

    kw = dict(kw)
    noise = kw.pop("noise", 0.0)
    items = []
    for pid, n in enumerate((N, big)):
        p = W.mixture_problem(700 + d + pid, d, 5, 5.0, lam_range=(0.1, 1.0), noise_sigma=noise)
        c = W.RunConfig(N=n, n_osc=4, n_conv=9, eps_grad=1e-3, seed=3, problem_id=pid, **kw)
        items.append((p, c, W.uniform_population(d + pid, n, p.lo, p.hi)))
    with Optimizer(*items[0]) as one, Optimizer.batched(items) as both:
        stats = [one.cycle(4, stats=True), [s[0] for s in both.cycle(4, stats=True)]]
        states = [_state(one), _state(both, 0)]
    assert stats[0] == stats[1]
    _assert_same(states[0], states[1], f"d={d}")


def test_closed_form_differences():
    from paper_2606_26164_amd.api import Optimizer

    items = []
    for pid, n in enumerate((300, 2100)):
        p = W.closed_form_problem("michalewicz", 7)
        c = W.RunConfig(N=n, n_osc=3, n_conv=8, eps_grad=1e-3, grad_mode=0, seed=4, problem_id=pid)
        items.append((p, c, W.uniform_population(1 + pid, n, p.lo, p.hi)))
    with Optimizer(*items[0]) as one, Optimizer.batched(items) as both:
        stats = [one.cycle(3, stats=True), [s[0] for s in both.cycle(3, stats=True)]]
        _assert_same(_state(one), _state(both, 0), "michalewicz")
    assert stats[0] == stats[1]
