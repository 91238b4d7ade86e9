"""The contraction in two f16 parts (d > 16) at the edges of its tiles, of its
dispatch rule and of f16's range, against the FP64 oracle.

Bounds are those of the float32 contraction, which it must not exceed: the
value is off by at most 64 u (|f| + max_k q_k / 2 + 1), u = 2^-24, and a
gradient by 1e-4 of its row's scale plus the value error times the largest
|P_k delta_k| where components compete."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle as O
from test_gpu_eval import _opt, _points, _value_bound

pytestmark = pytest.mark.gpu


def _check(prob, X, f, G, floor=1e-5):
    op = O.OracleProblem(prob)
    Xd = X.astype(np.float64)
    f_or, G_or = op.eval(Xd)
    fb, _ = _value_bound(f_or, Xd, op)
    assert np.all(np.abs(f - f_or) <= fb), float((np.abs(f - f_or) / fb).max())
    if G is None:
        return
    umax = np.zeros(len(Xd))
    for k in range(op.K):
        umax = np.maximum(umax, np.abs((Xd - op.mu[k]) @ op.prec[k]).max(1))
    gb = 1e-4 * np.abs(G_or).max(1) + floor + 4 * fb * (umax if op.K > 1 else 0.0)
    assert np.all(np.abs(G - G_or).max(1) <= gb), float((np.abs(G - G_or).max(1) / gb).max())


def _eval(prob, X, **kw):
    with _opt(prob) as opt:
        f, G = opt.eval(torch.from_numpy(np.ascontiguousarray(X, np.float32)).cuda(), **kw)
    return f.cpu().numpy().astype(np.float64), None if G is None else G.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("d,K,fam", [(17, 1, W.GAUSS), (17, 2, W.STUDENT_T), (31, 3, W.GAUSS), (32, 48, W.STUDENT_T),
                                     (33, 2, W.GAUSS), (63, 5, W.STUDENT_T), (64, 1, W.GAUSS)])
@pytest.mark.parametrize("B", [1, 16, 17, 33, 250])
def test_edges_of_tiles(d, K, fam, B):
    prob = W.mixture_problem(300 + d + K, d, K, 5.0, lam_range=(0.1, 1.0), family=fam, nu=3.0)
    X = _points(prob, max(B, 3), d)[:B]
    f, G = _eval(prob, X)
    _check(prob, X, f, G)
    f1, _ = _eval(prob, X, want_g=False)
    assert np.array_equal(f1, f)


@pytest.mark.parametrize("d", [20, 64])
def test_points_far_outside_the_box_and_non_finite_ones(d):
    """A far point carries a power of two of its own: nothing overflows that
    does not in float32, and its neighbours in the tile are as without it."""
    prob = W.mixture_problem(11, d, 6, 5.0, lam_range=(0.1, 1.0))
    near = _points(prob, 24, 3)
    f0, G0 = _eval(prob, near)
    u = np.random.default_rng(1).standard_normal((24, d))
    far = (10.0 ** np.linspace(1, 16, 24)[:, None] * u).astype(np.float32)
    X = np.empty((48, d), np.float32)
    X[0::2], X[1::2] = near, far
    f, G = _eval(prob, X)
    assert np.array_equal(f[0::2], f0) and np.array_equal(G[0::2], G0)
    # one component at a time decides a far point; the others' weights are 0
    _check(prob, far, f[1::2], None)
    G_or = O.OracleProblem(prob).eval(far.astype(np.float64))[1]
    rel = np.abs(G[1::2] - G_or).max(1) / np.abs(G_or).max(1)
    assert np.quantile(rel, 0.75) <= 1e-4, rel
    bad = near.copy()
    bad[3, d - 1], bad[7, 0], bad[20, 5] = np.nan, np.inf, 1e30
    f, G = _eval(prob, bad)
    rows = np.ones(24, bool)
    rows[[3, 7, 20]] = False
    assert not np.isfinite(f[~rows]).any()
    assert np.array_equal(f[rows], f0[rows]) and np.array_equal(G[rows], G0[rows])


@pytest.mark.parametrize("what", ["in", "span", "ratio", "scales"])
def test_either_side_of_the_rule(what):
    """A box of more than 2^10 standard deviations, or diagonals more than 2^12
    apart, stay in float32; coordinates of very different scale do not need to.
    Points 1e-4 standard deviations off a centre show a lost operand."""
    d, K = 24, 3
    prob = W.mixture_problem(12, d, K, 5.0, lam_range=(0.25, 1.0))
    if what == "span":
        prob.lo[:], prob.hi[:] = -4000.0, 4000.0
    if what == "ratio":
        prob.prec[0] = prob.prec[0] * np.float32(2.0 ** -14)
    if what == "scales":
        s = np.float32(2.0) ** np.linspace(-12, 12, d).round().astype(np.float32)
        prob.mu = prob.mu * s
        prob.lo, prob.hi = prob.lo * s, prob.hi * s
        prob.prec = prob.prec / (s[:, None] * s[None, :])
    rng = np.random.default_rng(5)
    std = 1.0 / np.sqrt(np.stack([np.diag(p) for p in prob.prec]))
    for size in (1e-4, 1.0):
        k = rng.integers(0, K, 40)
        X = (prob.mu[k] + size * std[k] * rng.standard_normal((40, d))).astype(np.float32)
        f, G = _eval(prob, X)
        op = O.OracleProblem(prob)
        f_or, G_or = op.eval(X.astype(np.float64))
        assert np.all(np.abs(f - f_or) <= _value_bound(f_or, X.astype(np.float64), op)[0])
        # in units of each coordinate's own standard deviation
        e, g = np.abs(G - G_or) * std[k], np.abs(G_or) * std[k]
        assert np.all(e.max(1) <= 1e-4 * g.max(1) + 2.0 ** -26), (e.max(1) / g.max(1)).max()


@pytest.mark.parametrize("N", [2048, 2049, 9000])
@pytest.mark.parametrize("d", [20, 64])
def test_population_evaluations_either_side_of_the_size_rule(d, N):
    """Values and gradients that Phase 1 leaves (line-search tiles, half and
    full ones) at the positions it leaves."""
    from paper_2606_26164_amd.api import Optimizer

    prob = W.mixture_problem(13, d, 9, 5.0, lam_range=(0.1, 1.0))
    cfg = W.RunConfig(N=N, n_osc=2, n_conv=2, eps_grad=1e-3)
    with Optimizer(prob, cfg, W.uniform_population(13, N, prob.lo, prob.hi)) as opt:
        opt.run_phases(1 << 1)
        st = opt.get_state()
    rows = np.random.default_rng(0).permutation(N)[:1500]
    _check(prob, st["X"][rows], st["F"][rows].astype(np.float64), st["G"][rows].astype(np.float64))
