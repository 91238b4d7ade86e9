"""Direct evaluations on either side of the sizes at which several waves share
a tile's components (128, 512 and 1024 tiles of 32 points), with fewer
components than waves among them, against the FP64 oracle.  Bounds as in
test_gpu_two_part."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_eval import _opt, _points
from test_gpu_two_part import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,fam", [(9, 1, W.GAUSS), (16, 7, W.STUDENT_T), (24, 9, W.GAUSS), (32, 33, W.STUDENT_T),
                                     (64, 3, W.GAUSS), (64, 20, W.STUDENT_T)])
@pytest.mark.parametrize("B", [1, 15, 4096, 4097, 16384, 16385, 32768, 32769])
def test_either_side_of_each_size(d, K, fam, B):
    prob = W.mixture_problem(500 + d + K, d, K, 5.0, lam_range=(0.1, 1.0), family=fam, nu=3.0)
    rng = np.random.default_rng(B)
    base = _points(prob, 600, d)
    at = rng.integers(0, 600, B)
    at[-1] = 599
    X = torch.from_numpy(base[at]).cuda()
    with _opt(prob) as opt:
        f, G = opt.eval(X)
        f1, _ = opt.eval(X, want_g=False)
        _, G1 = opt.eval(X, want_f=False)
    assert torch.equal(f, f1) and torch.equal(G, G1)
    f, G = f.cpu().numpy().astype(np.float64), G.cpu().numpy().astype(np.float64)
    # equal rows are equal wherever they stand
    first = np.full(600, -1)
    first[at[::-1]] = np.arange(B)[::-1]
    assert np.array_equal(f, f[first[at]]) and np.array_equal(G, G[first[at]])
    rows = first[first >= 0]
    _check(prob, base[at[rows]], f[rows], G[rows])


@pytest.mark.parametrize("d,K,fam", [(1, 8, W.GAUSS), (2, 7, W.STUDENT_T), (3, 31, W.GAUSS), (4, 32, W.STUDENT_T),
                                     (5, 65, W.GAUSS), (8, 130, W.GAUSS)])
@pytest.mark.parametrize("B", [1, 63, 65, 65536, 65537])
def test_small_mixtures(d, K, fam, B):
    """Either side of the sizes at which four waves share 64 points, with more
    components than one staged chunk among them."""
    test_either_side_of_each_size(d, K, fam, B)


@pytest.mark.parametrize("d", [3, 16, 40])
def test_a_nan_stays_in_its_row(d):
    prob = W.mixture_problem(21, d, 3, 5.0, lam_range=(0.1, 1.0))
    X = _points(prob, 40, 2)
    with _opt(prob) as opt:
        f0, G0 = opt.eval(torch.from_numpy(X).cuda())
        X[17, 1] = np.nan
        f, G = opt.eval(torch.from_numpy(X).cuda())
    rows = torch.arange(40, device="cuda") != 17
    assert not torch.isfinite(f[17]) and not torch.isfinite(G[17]).any()
    assert torch.equal(f[rows], f0[rows]) and torch.equal(G[rows], G0[rows])


def test_handle_free_evaluation_takes_the_same_path():
    from paper_2606_26164_amd.api import eval_static

    for d, B in ((40, 33), (40, 5000), (40, 20000), (6, 100), (6, 70000)):
        prob = W.mixture_problem(22, d, 12, 5.0, lam_range=(0.1, 1.0))
        X = torch.from_numpy(_points(prob, B, 4)).cuda()
        with _opt(prob) as opt:
            f, G = opt.eval(X)
        fs, Gs = eval_static(prob, X)
        assert torch.equal(f, fs) and torch.equal(G, Gs)
