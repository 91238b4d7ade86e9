"""Points next to a centre at 0, where float32 holds every digit of a small
distance: the contraction in two f16 parts may be no further off than the chain
of float32 multiply-adds it stands in for, in every kernel that takes it."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt
from test_gpu_two_part_rule import _chain, _matrix

pytestmark = pytest.mark.gpu


def _problem(d, half_width, fam=W.GAUSS):
    """A component at 0 and one at the edge of the box, whose weight at the
    points below is 0 in float32."""
    rng = np.random.default_rng(d)
    P = np.stack([_matrix(rng, d, "log", 10), _matrix(rng, d, "log", 10)]).astype(np.float32)
    mu = np.stack([np.zeros(d), np.full(d, 0.8 * half_width)]).astype(np.float32)
    return W.Problem(fam, d, 2, np.log(np.full(2, 0.5)).astype(np.float32), mu, P,
                     np.full(d, -half_width, np.float32), np.full(d, half_width, np.float32), nu=3.0 if fam else 0.0)


def _points(P, n, size, seed):
    A = np.linalg.cholesky(np.linalg.inv(P.astype(np.float64)))
    z = np.random.default_rng(seed).standard_normal((n, len(P)))
    return (size * z @ A.T).astype(np.float32)


def _compare(P, X, G, fam=W.GAUSS):
    Xd, Pd = X.astype(np.float64), P.astype(np.float64)
    exact, f32 = -Xd @ Pd, -_chain(P, X)
    extra = 0.0
    if fam == W.STUDENT_T:  # the weight (nu + d) / (nu + q): a reciprocal and two products more
        w = ((3.0 + len(P)) / (3.0 + np.einsum("ni,ij,nj->n", Xd, Pd, Xd)))[:, None]
        exact, f32, extra = exact * w, f32 * w, 2.0 ** -22
    keep = np.linalg.norm(exact, axis=1) > 0
    norm = np.linalg.norm(exact[keep], axis=1)
    got, ref = (np.linalg.norm(g[keep] - exact[keep], axis=1) / norm for g in (G, f32))
    got, ref = np.sqrt(np.mean(got ** 2)), np.sqrt(np.mean(ref ** 2))
    assert got <= 1.06 * ref + extra, f"{got:.3g} against {ref:.3g} of a float32 contraction"


# 64 to 16384 points: shared by 8 waves, by 4, alone; 70000: shared components at d = 64
@pytest.mark.parametrize("B", [64, 6000, 20000, 70000])
@pytest.mark.parametrize("half_width", [6.0, 100.0])
@pytest.mark.parametrize("d,fam", [(20, W.GAUSS), (24, W.STUDENT_T), (33, W.GAUSS), (64, W.GAUSS), (64, W.STUDENT_T)])
def test_direct_evaluations(d, fam, half_width, B):
    prob = _problem(d, half_width, fam)
    sizes = [1.0, 0.1, 1e-2, 1e-3, 1e-5, 1e-9]
    X = np.concatenate([_points(prob.prec[0], 400, s, i) for i, s in enumerate(sizes)])
    rows = np.random.default_rng(B).permutation(np.arange(max(B, len(X))) % len(X))[:B]  # sizes mixed within a tile
    with _opt(prob) as opt:
        f, G = opt.eval(torch.from_numpy(X[rows]).cuda())
        f1, _ = opt.eval(torch.from_numpy(X[rows]).cuda(), want_g=False)
    assert torch.equal(f, f1)
    G = G.cpu().numpy().astype(np.float64)
    for i in range(len(sizes)):
        pick = rows // 400 == i
        if pick.sum() >= 8:
            seen = G[pick]
            _compare(prob.prec[0], X[rows[pick]], seen, fam)
    # a point's bits do not hang on its neighbours in the tile
    order = np.argsort(rows, kind="stable")
    same = rows[order][1:] == rows[order][:-1]
    assert np.array_equal(G[order][1:][same], G[order][:-1][same])


@pytest.mark.parametrize("N", [2049, 9000])
@pytest.mark.parametrize("d", [24, 64])
def test_line_searches_of_a_population(d, N):
    from paper_2606_26164_amd.api import Optimizer

    prob = _problem(d, 6.0)
    x0 = _points(prob.prec[0], N, 1e-3, 5)
    cfg = W.RunConfig(N=N, n_osc=2, n_conv=2, eps_grad=1e-20)
    with Optimizer(prob, cfg, x0) as opt:
        opt.run_phases(1 << 1)
        st = opt.get_state()
    moved = np.any(st["X"] != x0, axis=1)
    assert moved.mean() > 0.9
    rows = np.flatnonzero(moved)[:1500]
    _compare(prob.prec[0], st["X"][rows], st["G"][rows].astype(np.float64))
