"""Rows at which the quadratic forms of some components overflow and others do
not: a component whose term is 2^-inf has no part in the sums, however many
waves share the components (component 0 does not overflow here)."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def _problem(d, K, fam, step):
    """Wide components (every third) and narrow ones with 2^step times their precision (near a multiple of the
    identity: no product in their forms is a large negative number, whose overflow would be a NaN of its own)."""
    prob = W.mixture_problem(40 + d, d, K, 5.0, lam_range=(0.9, 1.0), family=fam, nu=3.0)
    wide = np.arange(K) % 3 == 0
    prob.prec[wide] = prob.prec[wide] * np.float32(2.0 ** -step)
    return prob, wide


def _reference(prob, wide, X):
    X = X.astype(np.float64)
    l, u, s, qs = [], [], [], []
    for k in np.flatnonzero(wide):
        P, dl = prob.prec[k].astype(np.float64), X - prob.mu[k]
        uk = dl @ P
        q = (dl * uk).sum(1)
        logdet = np.linalg.slogdet(P)[1]
        l.append(prob.log_w[k] + 0.5 * logdet - 0.5 * q)
        u.append(uk)
        qs.append(q)
    l = np.stack(l) - 0.5 * prob.d * np.log(2 * np.pi)
    m = l.max(0)
    f = m + np.log(np.exp(l - m).sum(0))
    return f, -sum(np.exp(a - f)[:, None] * b for a, b in zip(l, u)), np.max(qs, 0)


@pytest.mark.parametrize("B", [1, 130, 4096, 4097, 16385, 32769, 65537])
@pytest.mark.parametrize("d,K,step", [(2, 20, 100), (8, 12, 100), (8, 130, 100), (12, 40, 100), (24, 2, 10), (24, 40, 10),
                                      (40, 2, 100), (64, 11, 10)])
@pytest.mark.parametrize("grad_mode", [1, 0])
def test_overflown_components_have_no_part(d, K, step, B, grad_mode):
    """Far points: 2^(128 - step) is the largest form of a wide component, and
    every narrow one's is infinite.  With step 10 the box and the precisions
    suit the two-part contraction."""
    prob, wide = _problem(d, K, W.GAUSS, step)
    rng = np.random.default_rng(d + K)
    z = rng.standard_normal((50, d))
    scale = np.array([1.5, 2.5, 4.0])[rng.integers(0, 3, 50)] * 2.0 ** 64  # narrow forms from 2^129 on
    X = (z / np.linalg.norm(z, axis=1)[:, None] * scale[:, None]).astype(np.float32)
    f_or, G_or, q = _reference(prob, wide, X)
    rows = np.arange(B) % 50
    with _opt(prob, N=128, grad_mode=grad_mode) as opt:
        f, G = opt.eval(torch.from_numpy(X[rows]).cuda(), grad_mode=grad_mode)
    f, G = f.cpu().numpy().astype(np.float64), G.cpu().numpy().astype(np.float64)
    fb = 64 * U32 * (np.abs(f_or) + 0.5 * q + 1.0)
    assert np.all(np.abs(f - f_or[rows]) <= fb[rows])
    # one wide component decides a far point (weights of the others underflow);
    # two that tie to rounding are left out
    l2 = np.sort(np.stack([-0.5 * np.einsum("ni,ij,nj->n", X.astype(np.float64) - prob.mu[k], prob.prec[k].astype(np.float64),
                                            X.astype(np.float64) - prob.mu[k]) for k in np.flatnonzero(wide)]), 0)
    clear = np.ones(50, bool) if len(l2) == 1 else l2[-1] - l2[-2] > 4 * fb
    err = np.abs(G - G_or[rows])
    if grad_mode == 1:
        tol = 1e-4 * np.abs(G_or).max(1, keepdims=True) * np.ones(d)
    else:
        tol = 2 * fb[:, None] / (2.0 ** -7 * np.maximum(1.0, np.abs(X))) + 1e-2 * np.abs(G_or).max(1, keepdims=True)
    ok = clear[rows]
    assert np.isfinite(G[ok]).all() and np.all(err[ok] <= tol[rows][ok])
