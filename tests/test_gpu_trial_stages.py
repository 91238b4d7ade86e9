"""Line-search trials after the first in one launch or in two stages: a problem
alone (its class below the limit) and in a batch whose class is above it gives
the same bits and counts the same evaluations."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch import _assert_same, _state

pytestmark = pytest.mark.gpu


# widths 8, 16, 32, 64; in place and with lists; one, two, three and all fifteen trials; central differences
@pytest.mark.parametrize("d,N,big,kw", [(2, 700, 65600, {}), (8, 17000, 50000, dict(ls_max=15)),
                                        (12, 300, 65300, dict(ls_max=3)), (16, 3000, 63000, dict(ls_max=2)),
                                        (20, 1500, 15000, {}), (32, 600, 15900, dict(ls_max=15)),
                                        (33, 500, 7800, {}), (64, 1100, 7200, dict(ls_max=4)),
                                        (10, 200, 65500, dict(grad_mode=0, ls_max=1))])
def test_merged_trials_equal_staged(d, N, big, kw):
    from paper_2606_26164_amd.api import Optimizer

    items = []
    for pid, n in enumerate((N, big)):
        p = W.mixture_problem(40 + pid, d, 5, 8.0, lam_range=(0.1, 1.0))
        c = W.RunConfig(**{**dict(N=n, m=6, n_osc=3, n_conv=8, M=4, eps_grad=1e-3, grad_mode=1, seed=6,
                                  problem_id=pid), **kw})
        items.append((p, c, W.uniform_population(50 + pid, n, p.lo, p.hi)))
    with Optimizer(*items[0]) as one, Optimizer.batched(items) as both:
        stats = [one.cycle(3, stats=True), [s[0] for s in both.cycle(3, stats=True)]]
        states = [_state(one), _state(both, 0)]
    assert stats[0] == stats[1]
    _assert_same(states[0], states[1], f"d={d}")
