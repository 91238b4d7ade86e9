"""Large launches at width 64, whose waves share a component's operands, give
the bits of the tiles they replace: either side of the size at which they
begin, with a ragged last tile, an odd probe count and noise."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt, _points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,fam", [(33, 3, W.GAUSS), (49, 1, W.STUDENT_T), (64, 20, W.GAUSS)])
@pytest.mark.parametrize("B", [65504, 65505, 65536 + 77])
def test_direct(d, K, fam, B):
    prob = W.mixture_problem(800 + d, d, K, 5.0, lam_range=(0.1, 1.0), family=fam, nu=3.0)
    base = torch.from_numpy(_points(prob, 500, d)).cuda()
    at = torch.arange(B, device="cuda") * 7 % 500
    X = base[at]
    X[B // 2, 3] = float("nan")
    with _opt(prob) as opt:
        f0, G0 = opt.eval(base[torch.arange(32768 + 32, device="cuda") * 7 % 500])  # one wave per tile
        f, G = opt.eval(X)
        f1, _ = opt.eval(X, want_g=False)
    rows = torch.arange(B, device="cuda") != B // 2
    assert torch.equal(f[rows], f0[:500].repeat(B // 500 + 1)[:B][rows])
    assert torch.equal(G[rows], G0[:500].repeat(B // 500 + 1, 1)[:B][rows])
    assert torch.equal(f1[rows], f[rows]) and not torch.isfinite(f[~rows]).any()


@pytest.mark.parametrize("d,M,N", [(64, 16, 4096), (50, 7, 17000), (64, 32, 2100)])
def test_probes_alone_and_in_a_batch(d, M, N):
    """A batch whose smoothing launches are large against handles of their own,
    whose are not all."""
    from paper_2606_26164_amd.api import Optimizer

    items = []
    for i in range(3):
        prob = W.mixture_problem(820 + d + i, d, 4, 5.0, lam_range=(0.1, 1.0))
        n = N - 37 * i
        items.append((prob, W.RunConfig(N=n, M=M, n_osc=3, n_conv=3, sigma=0.1, eps_grad=1e-3, problem_id=i),
                      W.uniform_population(i, n, prob.lo, prob.hi)))
    with Optimizer.batched(items) as opt:
        opt.cycle(2)
        batch = [opt.get_state(problem=p)["X"] for p in range(3)]
    for p, it in enumerate(items):
        with Optimizer(*it) as opt:
            opt.cycle(2)
            assert np.array_equal(opt.get_state()["X"], batch[p])
