"""Central differences of a mixture on caller memory: one contraction a
component, the stencils' quadratic forms from it."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle as O

pytestmark = pytest.mark.gpu

# around the widths, a single component and chunks of 64, whole and ragged tiles of 16 and 64 points, both splits
CASES = [(1, 1, W.GAUSS, 1), (2, 65, W.STUDENT_T, 63), (3, 7, W.GAUSS, 130), (8, 40, W.GAUSS, 65),
         (8, 130, W.STUDENT_T, 1000), (9, 1, W.STUDENT_T, 15), (16, 32, W.GAUSS, 17), (16, 5, W.GAUSS, 40001),
         (17, 3, W.GAUSS, 16), (31, 48, W.STUDENT_T, 33), (32, 9, W.GAUSS, 20000), (33, 5, W.GAUSS, 100),
         (64, 128, W.STUDENT_T, 50)]


@pytest.mark.parametrize("fd_h", [0.0, 0.125, 3.0])
@pytest.mark.parametrize("d,K,fam,B", CASES)
def test_gradient_matches_float64_differences(d, K, fam, B, fd_h):
    """Against differences of float64 values with the float32 stencil points.
    Each of the two values is off by no more than the float32 quadratic forms
    of the centre and of the point allow, 64 u (|f| + q / 2 + 1) with the
    larger q of the two (for a Student-t the weight of q is at most (nu + d) /
    (nu + q), times q less than nu + d); over 2 h."""
    from paper_2606_26164_amd.api import Optimizer

    prob = W.mixture_problem(300 + d, d, K, 5.0, lam_range=(0.1, 1.0), family=fam, nu=3.0)
    rng = np.random.default_rng(d + K)
    X = (prob.mu[rng.integers(0, K, B)] + rng.normal(0, 1.0, (B, d))).astype(np.float32)
    cfg = W.RunConfig(N=128, m=4, n_osc=2, grad_mode=0, eps_grad=1e-3, fd_h=fd_h, seed=1)
    with Optimizer(prob, cfg, W.uniform_population(1, cfg.N, prob.lo, prob.hi)) as opt:
        Xg = torch.from_numpy(X).cuda()
        f, G = opt.eval(Xg, grad_mode=0)
        f1, _ = opt.eval(Xg, grad_mode=0, want_g=False)
    assert torch.equal(f, f1)
    keep = np.unique(np.concatenate([np.arange(min(B, 40)), np.arange(max(0, B - 20), B)]))
    X, G = X[keep], G.cpu().numpy()[keep].astype(np.float64)
    h = (np.full_like(X, fd_h) if fd_h > 0 else np.ldexp(np.maximum(np.float32(1), np.abs(X)), -8)).astype(np.float32)
    up, dn = X + h, X - h
    op = O.OracleProblem(prob)

    def quad(Y):
        return np.stack([np.einsum("ni,ij,nj->n", Y - m, P, Y - m)
                         for m, P in zip(prob.mu.astype(np.float64), prob.prec.astype(np.float64))], 1)

    q0, u = quad(X.astype(np.float64)), 2.0 ** -24
    for j in range(d):
        side, bound = [], 0.0
        for z in (up, dn):
            Y = X.astype(np.float64)
            Y[:, j] = z[:, j]
            fy = op.eval(Y, grad=False)
            fy = fy[0] if isinstance(fy, tuple) else fy
            q = np.maximum(quad(Y), q0)
            # the components that carry the value at this point
            l = -0.5 * quad(Y) if fam == W.GAUSS else -0.5 * (3.0 + d) * np.log1p(quad(Y) / 3.0)
            w = l + prob.log_w
            carry = w >= w.max(1, keepdims=True) - 20.0
            weight = 0.5 if fam == W.GAUSS else 0.5 * (3.0 + d) / (3.0 + quad(Y))
            qc = np.where(carry, q * weight, 0.0).max(1)
            bound = bound + 64 * u * (np.abs(fy) + qc + 1.0)
            side.append(fy)
        den = up[:, j].astype(np.float64) - dn[:, j]
        ref = (side[0] - side[1]) / den
        err = np.abs(G[:, j] - ref)
        tol = bound / den + 1e-4 * np.abs(ref) + 1e-5
        assert np.all(err <= tol), f"coordinate {j}: error {err.max():.3g} of {tol.max():.3g}"


@pytest.mark.parametrize("d", [5, 16, 40])
def test_non_finite_points_stay_their_own(d):
    """A point with a NaN or an infinity gives no finite gradient and leaves
    the others as they are."""
    from paper_2606_26164_amd.api import Optimizer

    prob = W.mixture_problem(9, d, 6, 5.0, lam_range=(0.1, 1.0))
    cfg = W.RunConfig(N=128, m=4, n_osc=2, grad_mode=0, eps_grad=1e-3, seed=1)
    X = torch.from_numpy(W.uniform_population(2, 40, prob.lo, prob.hi)).cuda()
    Y = X.clone()
    Y[3, 0], Y[17, d - 1] = float("nan"), float("inf")
    with Optimizer(prob, cfg, W.uniform_population(1, cfg.N, prob.lo, prob.hi)) as opt:
        G, H = opt.eval(X, grad_mode=0)[1], opt.eval(Y, grad_mode=0)[1]
    rest = [i for i in range(40) if i not in (3, 17)]
    assert torch.equal(G[rest], H[rest])
    assert not torch.isfinite(H[[3, 17]]).any()
