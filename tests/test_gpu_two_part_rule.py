"""The contraction in two f16 parts is no further off than the float32 one it
stands in for, whatever the matrices: a chain of float32 multiply-adds over the
coordinates in order (the matrix core's float32 instruction) is emulated and its
error against float64 is what the library's may not exceed."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt

pytestmark = pytest.mark.gpu

ROWS = 300


def _matrix(rng, d, kind, c):
    if kind == "banded":
        a = rng.uniform(-0.9, 0.9, d - 1)
        return np.diag(rng.uniform(2.0, 4.0, d)) + np.diag(a, 1) + np.diag(a, -1)
    if kind == "blocks":
        p = np.eye(d)
        for i in range(0, d - 3, 4):
            b = rng.standard_normal((4, 4))
            p[i:i + 4, i:i + 4] += b @ b.T
        return p
    if kind == "weak":
        e = rng.standard_normal((d, d)) * 1e-3
        return np.diag(rng.uniform(1.0, 3.0, d)) + e + e.T
    lam = np.exp(rng.uniform(0.0, np.log(c), d)) if kind == "log" else np.r_[1.0 / c, np.ones(d - 1)]
    q = np.linalg.qr(rng.standard_normal((d, d)))[0] if c > 1 else np.eye(d)
    p = (q * lam) @ q.T
    return 0.5 * (p + p.T)


def _chain(P, D):
    acc = np.zeros(D.shape, np.float32)
    P64, D64 = P.astype(np.float64), D.astype(np.float64)
    for j in range(len(P)):
        acc = (acc + D64[:, j:j + 1] * P64[j:j + 1]).astype(np.float32)
    return acc.astype(np.float64)


def _ratio(d, kind, c, problems, power=0.5):
    """Error of the library's gradients over that of the chain, both against
    float64, at distances P^-power z, z normal.  One component, so that a
    gradient is -P delta."""
    rng = np.random.default_rng(d)
    got, ref = 0.0, 0.0
    for _ in range(problems):
        P = _matrix(rng, d, kind, c).astype(np.float32)
        mu = rng.uniform(-5.0, 5.0, (1, d)).astype(np.float32)
        prob = W.Problem(W.GAUSS, d, 1, np.zeros(1, np.float32), mu, P[None], np.full(d, -6.0, np.float32),
                         np.full(d, 6.0, np.float32))
        w, V = np.linalg.eigh(P.astype(np.float64))
        A = (V * w ** -power) @ V.T
        X = (mu + 1.5 * rng.standard_normal((ROWS, d)) @ A.T).astype(np.float32)
        with _opt(prob) as opt:
            G = opt.eval(torch.from_numpy(X).cuda())[1].cpu().numpy().astype(np.float64)
        exact = -(X.astype(np.float64) - mu) @ P.astype(np.float64)
        scale = np.linalg.norm(exact)
        got += (np.linalg.norm(G - exact) / scale) ** 2
        ref += (np.linalg.norm(-_chain(P, X - mu) - exact) / scale) ** 2
    return np.sqrt(got / ref)


@pytest.mark.parametrize("kind,c", [("log", 1), ("log", 3), ("log", 10), ("log", 100), ("log", 1e4), ("one", 100),
                                    ("one", 1e4), ("banded", 0), ("blocks", 0), ("weak", 0)])
@pytest.mark.parametrize("d", [17, 20, 24, 33, 49, 64])
def test_gradients_are_as_good_as_a_float32_contraction(d, kind, c):
    """6% for the scatter between 8 matrices' worth (a matrix's own rounding is
    a fixed error)."""
    assert _ratio(d, kind, c, 8) <= 1.06


@pytest.mark.parametrize("d", [24, 32, 33, 36, 40, 48, 52, 64])
def test_no_further_off_over_many_matrices(d):
    assert _ratio(d, "log", 10, 32) <= 1.0 + 1e-6  # (float32 itself where the rule takes it: the same sums)


@pytest.mark.parametrize("d", [28, 32, 36, 49, 52, 53, 64])
def test_no_further_off_at_the_end_of_an_ascent(d):
    """Distances along the small eigenvalues, where the steps of an ascent lead."""
    assert _ratio(d, "log", 10, 32, power=1.0) <= 1.0
