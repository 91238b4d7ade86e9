"""Central differences of a mixture whose steps are long beside a component:
centres many standard deviations away from a narrow component with a stencil
point next to its centre.  A quadratic form taken from the centre's loses all
of its digits there; the value of each stencil point has to be as good as one
evaluated on its own."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle as O
from test_gpu_eval import _opt

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def _quads(op, Y):
    return np.stack([np.einsum("ni,ij,nj->n", Y - m, P, Y - m) for m, P in zip(op.mu, op.prec)], 1)


@pytest.mark.parametrize("sd,fd_h", [(1e-2, 0.7), (1e-3, 3.0), (1e-4, 0.7), (1e-4, 3.0), (1e-2, 0.0)])
@pytest.mark.parametrize("d,K,fam,B", [(1, 2, W.STUDENT_T, 40), (2, 5, W.GAUSS, 70), (8, 3, W.STUDENT_T, 200),
                                       (8, 40, W.GAUSS, 65), (9, 2, W.GAUSS, 33), (16, 9, W.STUDENT_T, 17),
                                       (24, 1, W.GAUSS, 40), (32, 3, W.STUDENT_T, 16), (33, 4, W.GAUSS, 20),
                                       (64, 2, W.STUDENT_T, 40)])
def test_stencil_points_next_to_a_narrow_component(d, K, fam, B, sd, fd_h):
    """Against differences of float64 values at the float32 stencil points.  A
    value is off by at most 64 u (|f| + w q + 1) with q the largest form of the
    components that carry it, at the point itself, and w its weight in the log
    density (1/2, or (nu + d) / 2 / (nu + q)); a difference by both over 2 h."""
    prob = W.mixture_problem(900 + d + K, d, K, 5.0, lam_range=(0.1, 1.0), family=fam, nu=3.0)
    narrow = np.arange(K) % 2 == 0  # broad and narrow components mixed
    prob.prec[narrow] = prob.prec[narrow] * np.float32(sd ** -2)
    rng = np.random.default_rng(d + K)
    k, j = rng.choice(np.flatnonzero(narrow), B), rng.integers(0, d, B)
    near = prob.mu[k] + 0.3 * sd * rng.standard_normal((B, d))
    step = fd_h if fd_h > 0 else 2.0 ** -8 * np.maximum(1.0, np.abs(near[np.arange(B), j]))
    near[np.arange(B), j] -= step * rng.choice([-1.0, 1.0], B)  # one step away, to either side
    X = near.astype(np.float32)
    with _opt(prob, N=128, grad_mode=0, fd_h=fd_h) as opt:
        _, G = opt.eval(torch.from_numpy(X).cuda(), grad_mode=0)
    G = G.cpu().numpy().astype(np.float64)
    assert np.isfinite(G).all()
    h = (np.full_like(X, fd_h) if fd_h > 0 else np.ldexp(np.maximum(np.float32(1), np.abs(X)), -8)).astype(np.float32)
    up, dn = X + h, X - h
    op = O.OracleProblem(prob)
    for c in range(d):
        side, bound = [], 0.0
        for z in (up, dn):
            Y = X.astype(np.float64)
            Y[:, c] = z[:, c]
            q = _quads(op, Y)
            fy = op.eval(Y, grad=False)
            fy = fy[0] if isinstance(fy, tuple) else fy
            logdet = np.array([np.linalg.slogdet(P)[1] for P in op.prec])
            l = 0.5 * logdet + prob.log_w - (0.5 * q if fam == W.GAUSS else 0.5 * (3.0 + d) * np.log1p(q / 3.0))
            carry = l >= l.max(1, keepdims=True) - 20.0
            w = 0.5 if fam == W.GAUSS else 0.5 * (3.0 + d) / (3.0 + q)
            bound = bound + 64 * U32 * (np.abs(fy) + np.where(carry, w * q, 0.0).max(1) + 1.0)
            side.append(fy)
        den = up[:, c].astype(np.float64) - dn[:, c]
        ref = (side[0] - side[1]) / den
        err = np.abs(G[:, c] - ref)
        tol = bound / den + 16 * U32 * np.abs(ref)
        assert np.all(err <= tol), f"coordinate {c}: {(err / tol).max():.3g} of the bound"


@pytest.mark.parametrize("d", [2, 8, 12])
def test_a_component_whose_form_overflows_has_no_part(d):
    """q of the narrow component is infinite at the centres and at every stencil
    point; the broad one alone gives the gradient."""
    prob = W.mixture_problem(5, d, 2, 1.0, lam_range=(1.0, 1.0))
    both = dict(log_w=prob.log_w, mu=np.zeros((2, d), np.float32), lo=np.full(d, -1e15, np.float32),
                hi=np.full(d, 1e15, np.float32))
    for name, v in both.items():
        setattr(prob, name, v)
    prob.prec = np.stack([np.eye(d) * 1e-28, np.eye(d) * 1e12]).astype(np.float32)
    X = (1e14 * np.random.default_rng(1).standard_normal((20, d)) + 1e13).astype(np.float32)
    with _opt(prob, N=128, grad_mode=0) as opt:
        _, G = opt.eval(torch.from_numpy(X).cuda(), grad_mode=0)
    ref = -X.astype(np.float64) * 1e-28
    # f is of order q: its rounding over the distance of 2^-7 |x|
    assert np.all(np.abs(G.cpu().numpy() - ref) <= 64 * U32 * (0.5 * (X.astype(np.float64) ** 2).sum(1) * 1e-28 + 100)[:, None]
                  / (2.0 ** -7 * np.abs(X)) + 1e-6 * np.abs(ref))
