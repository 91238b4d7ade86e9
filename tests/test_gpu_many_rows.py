"""A call of more rows than one launch takes (2^29; HIP refuses 2^32 threads,
which four threads a row reach at 2^30 rows)."""
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grad_mode,K", [(1, 32), (0, 3)])
def test_rows_past_two_to_the_thirty(grad_mode, K):
    """d = 1: every launch's first and last rows have the bits of a call of
    their own of a size that takes the same kernel."""
    B = 2**30 + 65
    prob = W.mixture_problem(7, 1, K, 5.0, lam_range=(0.1, 1.0))
    g = torch.Generator(device="cuda").manual_seed(3)
    with _opt(prob) as opt:
        X = torch.rand(B, 1, generator=g, device="cuda").mul_(10.0).sub_(5.0)
        f, G = opt.eval(X, grad_mode=grad_mode)
        part = (B + 2) // 3  # 2^30 + 65 rows are three launches
        for at in (0, part, 2 * part):
            for lo in (at, min(at + part, B) - 70000):
                f1, G1 = opt.eval(X[lo:lo + 70000].clone(), grad_mode=grad_mode)
                assert torch.equal(f[lo:lo + 70000], f1) and torch.equal(G[lo:lo + 70000], G1)
