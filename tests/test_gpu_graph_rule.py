"""When a cycle is captured as a graph: with enough cycles of its kind left, or
after as many runs of it kernel by kernel on a handle that is set back.  Either
way every cycle gives bitwise the state of the same kernels enqueued one by
one, and every replay does."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch import _assert_same, _mixed_batch, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_osc", [4, 5, 7])  # never, exactly, amply enough cycles before the last
def test_batch_of_classes_across_the_capture_rule(n_osc):
    from paper_2606_26164_amd import _lib as L
    from paper_2606_26164_amd.api import Optimizer

    items = _mixed_batch(n_osc=n_osc)
    with Optimizer.batched(items) as a, Optimizer.batched(items, flags=L.FLAG_NO_GRAPH) as b:
        for k in range(n_osc):
            a.cycle(1)
            b.cycle(1)
            for p in range(len(items)):
                _assert_same(_state(a, p), _state(b, p), f"cycle {k}, problem {p}")


def test_set_back_handle_changes_to_replay():
    from paper_2606_26164_amd import _lib as L
    from paper_2606_26164_amd.api import Optimizer

    prob = W.mixture_problem(21, 6, 12, 10.0, lam_range=(0.1, 1.0))
    cfg = W.RunConfig(N=500, m=8, n_osc=3, n_conv=10, M=6, eps_grad=1e-3, grad_mode=1, seed=5)
    x0 = W.uniform_population(21, cfg.N, prob.lo, prob.hi)
    with Optimizer(prob, cfg, x0) as a, Optimizer(prob, cfg.with_(flags=L.FLAG_NO_GRAPH), x0) as b:
        for turn in range(7):  # the cycles before the last replay from the third turn on, the last from the fifth
            got = []
            for opt in (a, b):
                opt.set_state(X=np.roll(x0, turn, axis=0), k=0)
                opt.cycle(cfg.n_osc)
                got.append(_state(opt))
            _assert_same(got[0], got[1], f"turn {turn}")
