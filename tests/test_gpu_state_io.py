"""State transfer between dense host arrays and the library's padded rows."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _batch(N=(257, 1, 1000)):
    from paper_2606_26164_amd.api import Optimizer

    items = []
    for i, (d, n) in enumerate(zip((3, 33, 64), N)):  # rows 64 floats apart for all three
        prob = W.mixture_problem(400 + i, d, 3, 5.0, lam_range=(0.1, 1.0))
        items.append((prob, W.RunConfig(N=n, n_osc=3, seed=5, problem_id=i),
                      W.uniform_population(400 + i, n, prob.lo, prob.hi)))
    return items, Optimizer.batched(items)


def test_rows_come_back_as_they_were_given():
    items, opt = _batch()
    rng = np.random.default_rng(0)
    with opt:
        for p, (prob, cfg, x0) in enumerate(items):
            assert np.array_equal(opt.get_state(problem=p)["X"], x0)
        new = [(rng.uniform(prob.lo, prob.hi, (cfg.N, prob.d))).astype(np.float32) for prob, cfg, _ in items]
        wid = [rng.uniform(0.1, 2.0, x.shape).astype(np.float32) for x in new]
        new[0][5, 1] = np.nan
        for p, x in enumerate(new):
            opt.set_state(X=x, Wd=wid[p], wvalid=np.ones(len(x), np.uint8), problem=p)
        for p, x in enumerate(new):
            st = opt.get_state(history=True, problem=p)
            assert np.array_equal(st["X"], x, equal_nan=True) and np.array_equal(st["Wd"], wid[p])


def test_a_row_outside_the_box_is_named_and_nothing_is_written():
    from paper_2606_26164_amd import _lib as L
    from paper_2606_26164_amd.api import Optimizer

    items, opt = _batch()
    with opt:
        for p, (prob, cfg, x0) in enumerate(items):
            x = 0.5 * x0
            rows = sorted({cfg.N // 3, cfg.N - 1})
            for r in rows:
                x[r, prob.d - 1] = np.float32(prob.hi[-1]) * np.float32(1.0001)
            with pytest.raises(L.ChisaoError, match=f"sample {rows[0]} lies outside"):
                opt.set_state(X=x, problem=p)
            assert np.array_equal(opt.get_state(problem=p)["X"], x0)
    prob, cfg, x0 = items[1]
    for bad in (np.nan, np.inf, -7.0):
        x = x0.copy()
        x[0, 4] = bad
        with pytest.raises(L.ChisaoError, match="x0 sample 0 lies outside"):
            Optimizer(prob, cfg, torch.from_numpy(x).cuda())
