"""Workloads whose speed this library is held to, each one pass through its public entry points.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) the inputs and the handle a user's program holds before the call
    run(state)          one pass; returns its outputs
    work(case)          bytes and flops the pass cannot do without
    exact(case, seed)   the outputs in float64 (plain torch), where they have such values

Kinds of case
    eval     ``Optimizer.eval`` with the analytic gradient: values alone (``grad`` false) or values and gradients
    train    ``log_density`` forward and backward through torch autograd
    fd       ``Optimizer.eval`` with central differences (the plain path: 2 d evaluations a gradient)
    explore  the smoothing and anti-convergence phases of a cycle on a whole population, and its new positions
    polish   new candidate points into a handle that is kept, L-BFGS ascent, stick test and deduplication, and the
             polished points: a run's last cycle
    solve    a whole run from the problem to its modes, one problem or a batch of uneven ones

Points are what these calls meet once a search is under way: draws from the mixture's own components (``spread``
standard deviations wide).  Runs from a uniform start are the solve cases; they use the paper's own mixture, isotropic
components of equal weight, whose set of modes does not hang on the last bit of a sample's path.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2606_26164_amd import log_density
from paper_2606_26164_amd.api import Optimizer

GAUSS, STUDENT_T, MICHALEWICZ = 0, 1, 6
FD, ADJOINT = 0, 1


def listed():
    return [
        # One point at a time, as a sequential sampler or a line search in a caller's own loop asks for it: launch
        # latency and one pass over the components.
        dict(name="eval_one_point_d16", kind="eval", family=GAUSS, d=16, K=32, B=1, grad=True, spread=1.5),
        # A small batch of chains on the largest mixture: the chip is nearly empty, K components in a row.
        dict(name="eval_100_chains_d64", kind="eval", family=GAUSS, d=64, K=128, B=100, grad=True, spread=1.5),
        # Log densities alone, ragged in every size (20 of 32 coordinates, 7 components, an odd number of points).
        dict(name="density_student_d20", kind="eval", family=STUDENT_T, d=20, K=7, B=50021, grad=False, spread=2.0),
        # Low dimension, many points: one point per lane, no matrix product worth the name.
        dict(name="eval_d8_many", kind="eval", family=GAUSS, d=8, K=40, B=300000, grad=True, spread=2.0),
        # The largest batch: values and gradients of 262144 points of the d = 64, K = 128 mixture.
        dict(name="eval_d64_large", kind="eval", family=GAUSS, d=64, K=128, B=262144, grad=True, spread=1.5),
        # A torch model trained through the log density (forward and backward), Student-t, d = 32, K = 48.
        dict(name="train_student_d32", kind="train", family=STUDENT_T, d=32, K=48, B=8192, spread=2.0),
        # The central-difference path on the d = 16, K = 32 mixture with its population of 16384, at a fixed step of an
        # eighth: the default step, 2^-8 |x|, leaves float32 differences of these values good to 4e-5 only.
        dict(name="fd_d16", kind="fd", family=GAUSS, d=16, K=32, B=16384, spread=2.0, fd_h=0.125),
        # The same path on a closed-form test function, d = 64, at the default step.
        dict(name="fd_michalewicz_d64", kind="fd", family=MICHALEWICZ, d=64, K=0, B=8192, spread=1.0, fd_h=0.0),
        # Phases 5 and 6 of the headline workload (d = 64, K = 128, 65536 samples, 3 steps of 16 probes, 5 steps).
        dict(name="explore_d64", kind="explore", family=GAUSS, d=64, K=128, B=65536, M=16, spread=2.5),
        # Candidates from another search polished to maxima, d = 32: a run's last cycle on a kept handle.
        dict(name="polish_d32", kind="polish", family=GAUSS, d=32, K=48, B=8192, m=10, n_conv=15, spread=1.5),
        # A whole small run, the paper's population of a few hundred: many short launches, set-up included.
        dict(name="solve_d6_small", kind="solve", problems=1, d=6, K=6, B=256, M=10, m=5, n_osc=20),
        # A batch of uneven problems solved side by side.
        dict(name="solve_batch16", kind="solve", problems=16, d=64, K=32, B=4096, M=10, m=8, n_osc=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "eval", "train", "fd", "fd", "explore", "polish", "solve"])
    if kind == "solve":
        return dict(kind="solve", problems=rng.choice([1, 1, rng.randint(2, 16)]), d=rng.randint(2, 64),
                    K=rng.randint(2, 32), B=_log_int(rng, 200, 4096), M=rng.choice([4, 8, 10, 16]),
                    m=rng.choice([5, 8, 10]), n_osc=rng.randint(2, 20 if rng.random() < 0.5 else 4))
    c = dict(kind=kind, family=rng.choice([GAUSS, GAUSS, STUDENT_T]), spread=rng.choice([1.0, 1.5, 2.0, 2.5]))
    c["d"] = rng.choice([rng.randint(2, 64), rng.choice([2, 4, 8, 16, 32, 64])])
    c["K"] = _log_int(rng, 4, 128)
    if kind == "eval":
        c["B"] = _log_int(rng, 1, 262144)
        c["grad"] = rng.random() < 0.7
    elif kind == "train":
        c["B"] = _log_int(rng, 64, 65536)
    elif kind == "fd":
        c["d"] = rng.randint(2, 32)
        c["family"] = GAUSS
        c["K"] = _log_int(rng, 4, 64)
        c["B"] = _log_int(rng, 16, 16384)
        c["fd_h"] = 0.125
        if rng.random() < 0.3:
            c.update(family=MICHALEWICZ, d=rng.randint(2, 64), K=0, spread=1.0, fd_h=0.0)
    elif kind == "explore":
        c.update(d=rng.randint(4, 64), B=_log_int(rng, 1024, 65536), M=rng.choice([8, 10, 16]), spread=2.5)
    else:
        c.update(family=GAUSS, d=rng.randint(4, 64), B=_log_int(rng, 256, 8192), m=rng.choice([5, 8, 10]),
                 n_conv=rng.randint(12, 18), spread=1.5)
    return c


# ---- problems and points --------------------------------------------------------------------------------------------
def _mixture(g, family, d, K, mean_range, lam=(0.1, 1.0), iso=None):
    """Weights, centres and precision matrices Q diag(1 / lam) Q^T (Q Haar, lam log-uniform), or isotropic components
    of variance ``iso`` and equal weight."""
    mu = (torch.rand(K, d, generator=g, dtype=torch.float64) * 2 - 1) * mean_range
    if iso is None:
        lo, hi = math.log(lam[0]), math.log(lam[1])
        lv = torch.exp(lo + (hi - lo) * torch.rand(K, d, generator=g, dtype=torch.float64))
        q, r = torch.linalg.qr(torch.randn(K, d, d, generator=g, dtype=torch.float64))
        q = q * torch.sign(torch.diagonal(r, dim1=1, dim2=2))[:, None, :]
        w = torch.rand(K, generator=g, dtype=torch.float64) + 0.5
    else:
        lv = torch.full((K, d), float(iso), dtype=torch.float64)
        q = torch.eye(d, dtype=torch.float64).expand(K, d, d)
        w = torch.ones(K, dtype=torch.float64)
    p = (q / lv[:, None, :]) @ q.transpose(1, 2)
    p = 0.5 * (p + p.transpose(1, 2))
    a = np.full(d, 1.2 * mean_range, np.float32)
    prob = SimpleNamespace(family=family, d=d, K=K, log_w=torch.log(w / w.sum()).numpy().astype(np.float32),
                           mu=mu.numpy().astype(np.float32), prec=p.numpy().astype(np.float32), lo=-a, hi=a,
                           nu=3.0 if family == STUDENT_T else 0.0, noise_sigma=0.0)
    return prob, q * torch.sqrt(lv)[:, None, :]


def _problem(case, seed):
    g = torch.Generator().manual_seed(int(seed))
    if case["family"] == MICHALEWICZ:
        d = case["d"]
        z = np.zeros(0, np.float32)
        return SimpleNamespace(family=MICHALEWICZ, d=d, K=0, log_w=z, mu=z.reshape(0, d), prec=z.reshape(0, d, d),
                               lo=np.zeros(d, np.float32), hi=np.full(d, np.pi, np.float32), nu=0.0,
                               noise_sigma=0.0), None
    return _mixture(g, case["family"], case["d"], case["K"], 20.0 if case["d"] > 16 else 10.0)


def _points(case, seed, prob, factors):
    """Points of the case on the GPU: mu_k + spread * A_k z with k uniform, kept inside the box; uniform in the box
    for a closed form."""
    B, d = case["B"], case["d"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    if factors is None:
        return torch.rand(B, d, generator=g, device="cuda") * float(prob.hi[0])
    z = torch.randn(B, d, generator=g, device="cuda") * case["spread"]
    k = torch.randint(0, case["K"], (B,), generator=g, device="cuda")
    x = torch.empty_like(z)
    A = factors.to("cuda", torch.float32).contiguous()
    mu = torch.from_numpy(prob.mu).cuda()
    for j in range(case["K"]):
        i = torch.nonzero(k == j)[:, 0]
        x[i] = mu[j] + z[i] @ A[j].t()
    return x.clamp_(float(prob.lo[0]), float(prob.hi[0]))


def _config(N, **kw):
    """The library's usual settings (n_conv 0: chosen from d; sigma, alpha 0: chosen from the population)."""
    c = dict(N=N, m=10, n_osc=3, n_conv=0, n_anti=5, n_cloud=3, M=10, eps_grad=1e-3, eps_dup=1e-3,
             log_delta=math.log(0.1), momentum=0.9, alpha=0.0, sigma=0.0, sigma_c=0.1, grad_mode=ADJOINT, fd_h=0.0,
             ls_c1=1e-4, ls_max=10, curv_eps=1e-10, gate_reps=0, phase_mask=0x7E, seed=0, problem_id=0, flags=0)
    c.update(kw)
    return SimpleNamespace(**c)


def _solve_items(case, seed):
    """(problem, config, None) of each problem: sizes of the case for one problem, spread below them in a batch."""
    g = torch.Generator().manual_seed(int(seed))
    items = []
    for i in range(case["problems"]):
        d, K, N = case["d"], case["K"], case["B"]
        if case["problems"] > 1:
            d = [2, 4, 8, 16, 32, 64][(i + d) % 6]
            K = 2 + (7 * i + K) % max(case["K"] - 1, 1)
            N = max(200, N - (i * N) // (2 * case["problems"]))
        if d <= 4:
            K = min(K, 6)  # more peaks in so small a box run into one another
        prob, _ = _mixture(g, GAUSS, d, K, 10.0, iso=0.25)
        items.append((prob, _config(N, m=case["m"], n_osc=case["n_osc"], M=case["M"], seed=int(seed), problem_id=i),
                      None))
    return items


# ---- one pass -------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        return dict(kind=kind, items=_solve_items(case, seed))
    prob, factors = _problem(case, seed)
    X = _points(case, seed, prob, factors)
    s = dict(kind=kind, case=case)
    if kind in ("eval", "train", "fd"):
        s["opt"] = Optimizer(prob, _config(256, grad_mode=FD if kind == "fd" else ADJOINT,
                                           fd_h=case.get("fd_h", 0.0), seed=int(seed)))
        s["X"] = X.requires_grad_(kind == "train")
        if kind == "train":
            g = torch.Generator(device="cuda").manual_seed(int(seed) + 2)
            s["w"] = torch.randn(case["B"], generator=g, device="cuda")
    elif kind == "explore":
        s["opt"] = Optimizer(prob, _config(case["B"], M=case["M"], sigma=0.1, seed=int(seed)), X)
    else:
        s["opt"] = Optimizer(prob, _config(case["B"], m=case["m"], n_osc=1, n_conv=case["n_conv"], seed=int(seed)))
        s["X"] = X.cpu().numpy()
        s["stuck"] = np.zeros(case["B"], np.uint8)
        s["active"] = np.ones(case["B"], np.uint8)
    return s


def run(s):
    kind = s["kind"]
    if kind == "eval":
        f, G = s["opt"].eval(s["X"], want_g=s["case"]["grad"])
        return {"f": f, "G": G}
    if kind == "fd":
        f, G = s["opt"].eval(s["X"], grad_mode=FD)
        return {"f": f, "G": G}
    if kind == "train":
        X = s["X"]
        X.grad = None
        f = log_density(X, s["opt"])
        f.backward(s["w"])
        return {"f": f.detach(), "G": X.grad}
    if kind == "explore":
        s["opt"].run_phases((1 << 5) | (1 << 6))
        return {"X": s["opt"].get_state()["X"]}
    if kind == "polish":
        s["opt"].set_state(X=s["X"], stuck=s["stuck"], active=s["active"], k=0)
        s["opt"].cycle(1)
        st = s["opt"].get_state()
        return {"X": st["X"], "F": st["F"]}
    with Optimizer.batched(s["items"]) as opt:
        opt.cycle(s["items"][0][1].n_osc)
        out = {}
        for p in range(opt.P):
            m = opt.modes(p)
            order = np.argsort(m.X[:, 0])  # the library lists modes by sample index
            table = np.zeros((2 * opt.specs[p].K, opt.specs[p].d + 1), np.float32)  # a row a mode, then zeros
            n = min(len(order), len(table))
            table[:n, :-1], table[:n, -1] = m.X[order][:n], m.F[order][:n]
            out["modes%d" % p], out["n%d" % p] = table, len(order)
        return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _eval_flops(d, K):
    return K * (2 * d * d + 4 * d)


def work(case):
    kind, d, K, B = case["kind"], case["d"], case["K"], case["B"]
    if kind == "solve":
        b = fl = 0
        for prob, c, _ in _solve_items(case, 0):
            probes = (case["n_osc"] - 1) * (3 * case["M"] + 5)
            fl += c.N * _eval_flops(prob.d, prob.K) * (probes + 4 * case["n_osc"])
            b += 4 * (2 * c.N * prob.d * case["n_osc"] + prob.K * (prob.d ** 2 + prob.d + 1))
        return {"bytes": b, "flops": fl}
    tables = 4 * K * (d * d + d + 1)
    if kind == "eval":
        return {"bytes": 4 * B * (d + 1 + (d if case["grad"] else 0)) + tables, "flops": B * _eval_flops(d, K)}
    if kind == "train":
        return {"bytes": 4 * B * (4 * d + 2) + tables, "flops": B * (_eval_flops(d, K) + d)}
    if kind == "fd":
        # a stencil value differs from the centre's in one coordinate: one contraction, then a few operations for each
        # of the 2 d points and K components (about 40 for a closed form's changed term)
        fl = B * (_eval_flops(d, K) + 2 * d * K * 8) if K else B * 2 * d * 40
        return {"bytes": 4 * B * (2 * d + 1) + tables, "flops": fl}
    if kind == "explore":
        return {"bytes": 8 * B * d + tables, "flops": B * _eval_flops(d, K) * (3 * case["M"] + 5)}
    return {"bytes": 8 * B * d + tables, "flops": B * _eval_flops(d, K) * 8}


# ---- the same in float64 --------------------------------------------------------------------------------------------
def _exact_mixture(prob, X, grad):
    X = X.double()
    B, d, K = X.shape[0], prob.d, prob.K
    mu = torch.from_numpy(prob.mu).to(X.device).double()
    P = torch.from_numpy(prob.prec).to(X.device).double()
    logdet = torch.linalg.slogdet(P)[1]
    lw = torch.from_numpy(prob.log_w).to(X.device).double() + 0.5 * logdet
    nu = float(np.float32(prob.nu))
    if prob.family == GAUSS:
        lw = lw - 0.5 * d * math.log(2 * math.pi)
    else:
        lw = lw + math.lgamma(0.5 * (nu + d)) - math.lgamma(0.5 * nu) - 0.5 * d * math.log(nu * math.pi)

    def component(k):
        dl = X - mu[k]
        u = dl @ P[k]
        q = (dl * u).sum(1)
        if prob.family == GAUSS:
            return u, lw[k] - 0.5 * q, None
        return u, lw[k] - 0.5 * (nu + d) * torch.log1p(q / nu), (nu + d) / (nu + q)

    logs = torch.empty(K, B, dtype=torch.float64, device=X.device)
    for k in range(K):
        logs[k] = component(k)[1]
    f = torch.logsumexp(logs, 0)
    if not grad:
        return f, None
    G = torch.zeros(B, d, dtype=torch.float64, device=X.device)
    for k in range(K):
        u, l, s = component(k)
        r = torch.exp(l - f)
        G -= (r if s is None else r * s)[:, None] * u
    return f, G


def _steps(X, fd_h):
    """The central-difference points of a coordinate, as float32 holds them: h = 2^-8 max(1, |x|), or the one given."""
    h = torch.clamp(X.abs(), min=1.0) * 2.0 ** -8 if fd_h <= 0 else fd_h
    return X + h, X - h


def _exact_fd(prob, X, fd_h):
    xp, xm = _steps(X, fd_h)
    if prob.family == MICHALEWICZ:
        i = torch.arange(1, prob.d + 1, device=X.device, dtype=torch.float64)

        def term(x):
            x = x.double()
            return torch.sin(x) * torch.sin(i * x * x / math.pi) ** 20

        return term(X).sum(1), (term(xp) - term(xm)) / (xp.double() - xm.double())
    f, _ = _exact_mixture(prob, X, False)
    G = torch.empty(X.shape, dtype=torch.float64, device=X.device)
    for j in range(prob.d):
        side = []
        for x in (xp, xm):
            Y = X.clone()
            Y[:, j] = x[:, j]
            side.append(_exact_mixture(prob, Y, False)[0])
        G[:, j] = (side[0] - side[1]) / (xp[:, j].double() - xm[:, j].double())
    return f, G


def exact(case, seed):
    kind = case["kind"]
    if kind in ("explore", "polish", "solve"):
        return None  # where a search stands after so many steps has no value of its own
    prob, factors = _problem(case, seed)
    X = _points(case, seed, prob, factors)
    if kind == "fd":
        f, G = _exact_fd(prob, X, case["fd_h"])
        return {"f": f, "G": G}
    f, G = _exact_mixture(prob, X, kind == "train" or case["grad"])
    if kind == "train":
        g = torch.Generator(device="cuda").manual_seed(int(seed) + 2)
        G = G * torch.randn(case["B"], generator=g, device="cuda").double()[:, None]
    return {"f": f, "G": G}
