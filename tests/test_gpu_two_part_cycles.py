"""Populations that contract in two f16 parts (d >= 24, more than 2048 samples)
against the FP64 oracle, phase by phase from the GPU's own states and decisions,
in the protocol and with the tolerances of the smaller populations' tests."""
import numpy as np
import pytest

import workloads as W
from oracle import oracle as O
from test_gpu_headline import _lbfgs_iteration_parity, _phase_states, _resumed
from test_gpu_phases import REPLAY, _gpu, _oracle_from, _rows_close

pytestmark = pytest.mark.gpu


def _d40():
    prob = W.mixture_problem(71, 40, 12, 6.0, lam_range=(0.1, 1.0))
    cfg = W.RunConfig(N=2304, m=8, n_osc=4, n_conv=14, M=8, sigma=0.1, eps_grad=1e-3, grad_mode=1, seed=8)
    return prob, cfg, W.uniform_population(71, 2304, prob.lo, prob.hi)


# 4096 samples of 16 probes: the probe launch shares components (2048 tiles)
CASES = [("gauss128_d64", lambda: W.gauss128_d64(N=4096, n_osc=4), 2),
         ("gauss12_d40", _d40, 3), ("student48_d32", lambda: W.student48_d32(N=2304, n_osc=4), 2)]


@pytest.mark.parametrize("name,make,cycles", CASES, ids=[c[0] for c in CASES])
def test_every_phase_matches_oracle(name, make, cycles):
    prob, cfg, x0 = make()
    op = O.OracleProblem(prob)
    span = float((prob.hi - prob.lo).max())
    with _gpu(prob, cfg, x0) as opt:
        starts = []
        for _ in range(cycles):
            starts.append(opt.get_state(history=True))
            opt.cycle(1)
    for k, s0 in enumerate(starts):
        for t in (1, 5, cfg.n_conv - 1):
            n_moved, e = _lbfgs_iteration_parity(op, prob, cfg, s0, t)
            print(f"\n{name} cycle {k + 1} iteration {t + 1}: {n_moved} moved, X relative error {e:.2e}")
        ph = _phase_states(prob, cfg, s0)
        # values and gradients are those of the GPU's own positions
        some = np.flatnonzero(ph["p1"]["active"])[:800]
        f, G = op.eval(ph["p1"]["X"][some].astype(np.float64))
        if not prob.noise_sigma > 0:
            _rows_close(ph["p1"]["F"][some][:, None], f[:, None], 1e-5, "F after phase 1")
        _rows_close(ph["p1"]["G"][some], G, 1e-4, "G after phase 1", floor=1.0)
        run = _oracle_from(op, cfg, ph["p1"])
        assert run.phase_stick(stuck_in=ph["p3"]["stuck_pre"], **REPLAY).n_hard == 0
        assert run.phase_dedup(removed_in=ph["p3"]["removed"], **REPLAY).n_hard == 0
        np.testing.assert_array_equal(run.stuck, ph["p3"]["stuck"])
        run.phase_reseed()
        assert np.abs(ph["p4"]["X"].astype(np.float64) - run.X).max() <= 2e-5 * span
        c1 = cfg.with_(n_cloud=1)
        with _resumed(prob, c1, ph["p4"]) as h:
            h.run_phases(1 << 5)
            g5 = h.get_state()
        run = _oracle_from(op, c1, ph["p4"])
        run.phase_hlc()
        _rows_close(g5["X"], run.X, 1e-4, "first smoothing step")
        run = _oracle_from(op, cfg, ph["p5"])
        run.st.sigma = cfg.sigma
        run.phase_anti()
        _rows_close(ph["p6"]["X"], run.X, 1e-4, "anti-convergence")


U32 = 2.0 ** -24


@pytest.mark.parametrize("fd_h", [0.0, 0.125])
@pytest.mark.parametrize("d,fam", [(24, W.GAUSS), (32, W.STUDENT_T), (40, W.GAUSS), (64, W.STUDENT_T)])
def test_central_differences_of_a_population(d, fam, fd_h):
    """Gradients after a first iteration, at the positions it leaves, against
    differences of float64 values at the float32 stencil points.  A value is off
    by 64 u (|f| + q / 2 + 1) at most (q the largest form), and 4 u of it in the
    root mean square, as in float32."""
    from paper_2606_26164_amd.api import Optimizer

    prob = W.mixture_problem(13, d, 9, 5.0, lam_range=(0.1, 1.0), family=fam, nu=3.0)
    rng = np.random.default_rng(d)
    N = 2304
    x0 = np.clip(prob.mu[rng.integers(0, 9, N)] + rng.normal(0, 0.6, (N, d)), prob.lo, prob.hi).astype(np.float32)
    cfg = W.RunConfig(N=N, n_osc=2, n_conv=1, eps_grad=1e-3, grad_mode=0, fd_h=fd_h)
    with Optimizer(prob, cfg, x0) as opt:
        opt.run_phases(1 << 1)
        st = opt.get_state()
    assert np.any(st["X"] != x0, axis=1).mean() > 0.9
    X, G = st["X"][:200], st["G"][:200].astype(np.float64)
    op = O.OracleProblem(prob)
    h = (np.full_like(X, fd_h) if fd_h > 0 else np.ldexp(np.maximum(np.float32(1), np.abs(X)), -8)).astype(np.float32)
    up, dn = X + h, X - h
    q = np.max([np.einsum("ni,ij,nj->n", X - m, P, X - m) for m, P in zip(op.mu, op.prec)], 0)
    off = []
    for j in range(d):
        side = []
        for z in (up, dn):
            Y = X.astype(np.float64)
            Y[:, j] = z[:, j]
            f = op.eval(Y, grad=False)
            side.append(f[0] if isinstance(f, tuple) else f)
        den = up[:, j].astype(np.float64) - dn[:, j]
        off.append(np.abs(G[:, j] - (side[0] - side[1]) / den) * den / (np.abs(side[0]) + 0.5 * q + 1.0))
    off = np.array(off)
    assert off.max() <= 2 * 64 * U32 and np.sqrt((off ** 2).mean()) <= np.sqrt(2.0) * 4 * U32, off.max() / U32


@pytest.mark.parametrize("d", [24, 40])
def test_smoothing_with_central_differences(d):
    """The first smoothing step of a central-difference population (stencils
    around its probes), tolerance as for the smaller populations."""
    prob = W.mixture_problem(51, d, 12, 5.0, lam_range=(0.2, 1.0))
    cfg = W.RunConfig(N=2304, m=6, n_osc=4, n_conv=12, n_cloud=1, M=4, sigma=0.3, eps_grad=1e-3, grad_mode=0, seed=6)
    with _gpu(prob, cfg, W.uniform_population(51, cfg.N, prob.lo, prob.hi)) as opt:
        g0 = opt.get_state()
        opt.run_phases(1 << 5)
        g5 = opt.get_state()
    run = _oracle_from(prob, cfg, g0)
    run.phase_hlc()
    got, want = g5["X"].astype(np.float64) - g0["X"], run.X - g0["X"]
    r = _rows_close(got, want, 5e-3, "smoothing displacement", floor=1e-3)
    print(f"\nd={d}: displacement relative error max {r.max():.2e}")
