"""Every form of X that ``Optimizer.eval`` takes gives the bits of the plain one."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt, _points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["double", "transposed", "strided", "flat", "three", "host", "leaf", "half"])
@pytest.mark.parametrize("d", [3, 20])
def test_forms_of_x(form, d):
    prob = W.mixture_problem(600 + d, d, 5, 5.0, lam_range=(0.1, 1.0))
    x = torch.from_numpy(_points(prob, 60, 1)).cuda()
    if form == "half":
        x = x.half().float()
    with _opt(prob) as opt:
        f0, G0 = opt.eval(x)
        y = {"double": lambda: x.double(), "transposed": lambda: x.t().contiguous().t(),
             "strided": lambda: torch.cat([x, x], 1)[:, :d], "flat": lambda: x.reshape(-1),
             "three": lambda: x.reshape(6, 10, d), "host": lambda: x.cpu(),
             "leaf": lambda: x.clone().requires_grad_(True), "half": lambda: x.half()}[form]()
        f, G = opt.eval(y)
        assert type(f) is torch.Tensor and not f.requires_grad and f.shape == (60,) and G.shape == (60, d)
        assert torch.equal(f, f0) and torch.equal(G, G0)
        f, G = opt.eval(y, want_f=False)
        assert f is None and torch.equal(G, G0)
        f, G = opt.eval(y, grad_mode=0, want_g=False)
        assert G is None and torch.equal(f, f0)


def test_backward_in_other_types_and_twice():
    from paper_2606_26164_amd import log_density

    prob = W.mixture_problem(8, 20, 4, 5.0, lam_range=(0.1, 1.0))
    x = torch.from_numpy(_points(prob, 33, 9)).cuda().requires_grad_(True)
    w = torch.linspace(-1, 2, 33, device="cuda")
    with _opt(prob) as opt:
        G = opt.eval(x)[1]
        f = log_density(x, opt)
        for _ in range(2):
            (g,) = torch.autograd.grad((f * w).sum(), x, retain_graph=True)
            assert torch.equal(g, w[:, None] * G)
        (g,) = torch.autograd.grad(log_density(x, opt).double().sum(), x)
        assert torch.equal(g, G)
