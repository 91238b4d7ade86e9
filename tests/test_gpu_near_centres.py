"""Points next to a centre at 0, where float32 holds every digit of a small
distance: the contraction in two f16 parts may be no further off there than a
standard deviation away, relative to the gradient, in every kernel that takes
it."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt
from test_gpu_two_part_rule import _chain, _matrix

pytestmark = pytest.mark.gpu


def _problem(d, half_width, seed=0):
    """A Gaussian component at 0 (a gradient is -P x: no weight of its own
    rounding) and one at the edge of the box, whose weight at the points below
    is 0 in float32."""
    rng = np.random.default_rng(100 * seed + d)
    P = np.stack([_matrix(rng, d, "log", 10), _matrix(rng, d, "log", 10)]).astype(np.float32)
    mu = np.stack([np.zeros(d), np.full(d, 0.8 * half_width)]).astype(np.float32)
    return W.Problem(W.GAUSS, d, 2, np.log(np.full(2, 0.5)).astype(np.float32), mu, P,
                     np.full(d, -half_width, np.float32), np.full(d, half_width, np.float32))


def _points(P, n, size, seed):
    A = np.linalg.cholesky(np.linalg.inv(P.astype(np.float64)))
    z = np.random.default_rng(seed).standard_normal((n, len(P)))
    return (size * z @ A.T).astype(np.float32)


def _error(P, X, G):
    """Relative 2-norm error of a row, root mean square over the rows."""
    Xd, Pd = X.astype(np.float64), P.astype(np.float64)
    exact = -Xd @ Pd
    norm = np.linalg.norm(exact, axis=1)
    keep = norm > 0
    return np.sqrt(np.mean((np.linalg.norm(G[keep] - exact[keep], axis=1) / norm[keep]) ** 2))


# 20% for the scatter of a mean over few rows; an f16 part that ran out of bits shows as a factor of 3 and more
SCATTER = 1.2


# up to 16384 points: shared by 8 waves, by 4, alone; 70000: shared components at d = 64
@pytest.mark.parametrize("B", [300, 6000, 20000, 70000])
@pytest.mark.parametrize("half_width", [6.0, 100.0])
@pytest.mark.parametrize("d", [20, 24, 33, 64])
def test_direct_evaluations(d, half_width, B):
    prob = _problem(d, half_width)
    sizes = [1.0, 0.1, 1e-2, 1e-3, 1e-5, 1e-9]
    X = np.concatenate([_points(prob.prec[0], 400, s, i) for i, s in enumerate(sizes)])
    rows = np.random.default_rng(B).permutation(np.arange(max(B, len(X))) % len(X))[:B]  # sizes mixed within a tile
    with _opt(prob) as opt:
        f, G = opt.eval(torch.from_numpy(X[rows]).cuda())
        f1, _ = opt.eval(torch.from_numpy(X[rows]).cuda(), want_g=False)
    assert torch.equal(f, f1)
    G = G.cpu().numpy().astype(np.float64)
    err = [_error(prob.prec[0], X[rows[rows // 400 == i]], G[rows // 400 == i]) for i in range(len(sizes))]
    assert max(err) <= SCATTER * err[0], err
    # a point's bits do not hang on its neighbours in the tile
    order = np.argsort(rows, kind="stable")
    same = rows[order][1:] == rows[order][:-1]
    assert np.array_equal(G[order][1:][same], G[order][:-1][same])


@pytest.mark.parametrize("N", [2049, 9000])
@pytest.mark.parametrize("d", [24, 40, 64])
def test_line_searches_of_a_population(d, N):
    """Where the steps led, next to the centre, sums cancel more than at random
    points: against a chain of float32 multiply-adds there, over 6 matrices."""
    from paper_2606_26164_amd.api import Optimizer

    err, f32 = [], []
    for seed in range(6):
        prob = _problem(d, 6.0, seed)
        x0 = _points(prob.prec[0], N, 1e-3, 5)
        cfg = W.RunConfig(N=N, n_osc=2, n_conv=2, eps_grad=1e-20)
        with Optimizer(prob, cfg, x0) as opt:
            opt.run_phases(1 << 1)
            st = opt.get_state()
        moved = np.any(st["X"] != x0, axis=1)
        assert moved.mean() > 0.9
        X, G = (st[k][np.flatnonzero(moved)[:500]] for k in ("X", "G"))
        assert np.abs(X).max() < 1e-2
        err.append(_error(prob.prec[0], X, G.astype(np.float64)))
        f32.append(_error(prob.prec[0], X, -_chain(prob.prec[0], X)))
    assert np.mean(err) <= SCATTER * np.mean(f32), (err, f32)
