"""The work that programs have this library do, as cases that can be timed.

A case is one whole call (or one short sequence of calls) through the public
binding `paper_2110_11738_amd.drot`, on inputs a program would hold on the
GPU.  Four kinds:

  solve   one optimal-transport problem for a fixed number of iterations
          (tol = 0), from X_0 = p q^T or a warm start, to the plan, the duals
          and the objective.  Dense, bfloat16 or coordinate cost.
  batch   many problems of different shapes in one call.
  grid    many histogram pairs on one grid (one shared cost): the warm start's
          training data, of which the program keeps the duals.
  mlp     the warm-start network: a forward pass, or loss and gradients.

A solve to a tolerance takes 10^3 to 10^5 iterations of the same work; the
iteration counts here (up to the 1000 of the paper's accuracy experiment) keep
a pass short.  Duals and objectives of float32 problems are handed on in
float32, as the warm start's training does with its targets.
"""
import math

import numpy as np
import torch

from paper_2110_11738_amd import drot

DEV = "cuda"


def listed():
    return [
        # The smallest problems, where one iteration is microseconds: the
        # paper's smallest runtime size, and the float64 accuracy experiment.
        dict(name="solve_f32_100", kind="solve", cost="f32", m=100, n=100, iters=1000),
        dict(name="solve_f64_100", kind="solve", cost="f64", m=100, n=100, iters=1000),
        # Ordinary problems of a few hundred to a thousand points a side, odd
        # sizes with a plain contiguous cost matrix, in both types.
        dict(name="solve_f32_517x483", kind="solve", cost="f32", m=517, n=483, iters=1000,
             padded=False),
        dict(name="solve_f64_700x901", kind="solve", cost="f64", m=700, n=901, iters=300),
        # A middle size of the paper's runtime experiment.
        dict(name="solve_f32_2000", kind="solve", cost="f32", m=2000, n=2000, iters=300),
        # The headline workload: 4096^2, mixtures of Gaussians.
        dict(name="solve_f32_4096", kind="solve", cost="f32", m=4096, n=4096, iters=200),
        # The largest size of the paper's runtime experiment.
        dict(name="solve_f32_20000", kind="solve", cost="f32", m=20000, n=20000, iters=16),
        # The precision workload's cheaper costs: points in the unit cube.
        dict(name="solve_coords_10000x15000", kind="solve", cost="coords", dim=3, m=10000,
             n=15000, iters=32),
        dict(name="solve_bf16_10000x15000", kind="solve", cost="bf16", dim=3, m=10000, n=15000,
             iters=32),
        # A batch of ragged problems, sides uniform in [64, 2048].
        dict(name="batch_ragged_20", kind="batch", count=20, lo=64, hi=2048, shapes=0, iters=100),
        # Training data of the warm start: 128 pairs of 32 x 32 histograms.
        dict(name="grid_32_128", kind="grid", side=32, count=128, iters=100),
        # One mini-batch of the warm start's training, forward and backward.
        dict(name="mlp_gradients_256", kind="mlp", inp=2048, hidden=512, out=2048, batch=256,
             op="gradients"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("solve", "batch", "grid", "mlp"), (12, 2, 1, 3))[0]
    if kind == "solve":
        cost = rng.choices(("f32", "f64", "bf16", "coords"), (6, 3, 2, 2))[0]
        m, n = _log_int(rng, 8, 20000), _log_int(rng, 8, 20000)
        if rng.random() < 0.4:  # nearly square, as most problems are
            n = min(20000, max(8, int(m * rng.uniform(0.8, 1.25))))
        if cost == "f64":
            m, n = min(m, 9000), min(n, 9000)
        iters = max(8, min(1000, int(3e9 / (m * n))))
        case = dict(kind=kind, cost=cost, m=m, n=n, iters=iters, padded=rng.random() < 0.6)
        if cost == "coords":
            case["dim"] = rng.choice((1, 2, 3))
        if rng.random() < 0.2:
            case["warm"] = True
        if cost == "f32" and rng.random() < 0.25:
            case["option"] = rng.choice(("compensated", "skip_c"))
        return case
    if kind == "batch":
        lo = _log_int(rng, 16, 512)
        return dict(kind=kind, count=rng.randint(2, 20), lo=lo, hi=rng.randint(lo + 64, 2048),
                    shapes=rng.randint(1, 10 ** 6), iters=rng.randint(20, 100))
    if kind == "grid":
        return dict(kind=kind, side=rng.randint(8, 32), count=rng.randint(8, 128),
                    iters=rng.randint(20, 100))
    return dict(kind=kind, inp=64 * rng.randint(2, 32), hidden=64 * rng.randint(1, 16),
                out=64 * rng.randint(2, 32), batch=64 * rng.randint(1, 8),
                op=rng.choice(("forward", "gradients")))


# ---------------------------------------------------------------------------
# Inputs, from the seed alone.
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _marginal(w):
    """Weights as a probability vector on a dyadic grid: entries of at most 23
    bits and a sum of exactly 1, in float32 and in float64."""
    w = w / w.sum()
    e = torch.floor(torch.log2((2.0 ** 22) / w.max())).clamp(max=60.0)
    one = torch.exp2(e)
    k = torch.round(w * one)
    k[torch.argmax(k)] += one - k.sum()
    return k / one


def _mixture(g, k, d, comps=5, sigma=0.1):
    means = _rand(g, comps, d)
    comp = torch.randint(0, comps, (k,), generator=g, device=DEV)
    return means[comp] + sigma * torch.randn(k, d, generator=g, device=DEV, dtype=torch.float64)


def _sq_cost(xs, xt, dtype):
    """Squared distances over their maximum, in row blocks, rounded once."""
    m, n = xs.shape[0], xt.shape[0]
    C = torch.empty(m, n, dtype=dtype, device=DEV)
    blk = max(1, (1 << 25) // n)
    top = torch.zeros((), dtype=torch.float64, device=DEV)
    for last in (False, True):
        for i in range(0, m, blk):
            d = torch.zeros(min(blk, m - i), n, dtype=torch.float64, device=DEV)
            for k in range(xs.shape[1]):
                d += (xs[i:i + blk, k:k + 1] - xt[:, k]) ** 2
            if last:
                C[i:i + blk] = d / top
            else:
                top = torch.maximum(top, d.max())
    return C


def _problem(case, seed):
    """One problem of kind `solve`: the arrays the library is given."""
    g = _gen(seed)
    m, n, cost = case["m"], case["n"], case["cost"]
    dt = torch.float64 if cost == "f64" else torch.float32
    dim = case.get("dim", 2)
    if "dim" in case:  # points uniform in the unit cube
        xs, xt = _rand(g, m, dim), _rand(g, n, dim)
    else:
        xs, xt = _mixture(g, m, dim), _mixture(g, n, dim)
    p = _marginal(-torch.log1p(-_rand(g, m))).to(dt)
    q = _marginal(-torch.log1p(-_rand(g, n))).to(dt)
    out = dict(p=p, q=q, rho=(1.0 / math.log(max(m, 3))) / (m + n), mu0=None, nu0=None)
    if cost == "coords":
        out["xs"], out["xt"] = xs.float().contiguous(), xt.float().contiguous()
    else:
        out["C"] = _sq_cost(xs, xt, torch.bfloat16 if cost == "bf16" else dt)
    if case.get("warm"):
        out["mu0"] = 0.1 * torch.randn(m, generator=g, device=DEV, dtype=torch.float64)
        out["nu0"] = 0.1 * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    return out


def _batch_problems(case, seed):
    r = np.random.default_rng([4, case["shapes"]])
    sizes = r.integers(case["lo"], case["hi"] + 1, (case["count"], 2))
    probs = []
    for b, (m, n) in enumerate(sizes.tolist()):
        c = dict(cost="f32", m=m, n=n)
        probs.append(_problem(c, int(seed) * 1000 + b))
    return probs


def _histogram(g, side):
    """A histogram of 1 to 4 Gaussian bumps on a side x side grid."""
    ax = torch.arange(side, dtype=torch.float64, device=DEV)
    u = _rand(g, 4, 5)
    h = torch.zeros(side, side, dtype=torch.float64, device=DEV)
    bumps = 1 + int(torch.randint(0, 4, (1,), generator=g, device=DEV))
    for cx, cy, w, a, _ in u[:bumps].tolist():
        d2 = (ax[:, None] - side * cx) ** 2 + (ax - side * cy) ** 2
        h += (0.5 + a) * torch.exp(-d2 / (2 * (1 + 5 * w) ** 2))
    return _marginal(h.flatten())


def _grid_problems(case, seed):
    side, g = case["side"], _gen(seed)
    ax = torch.arange(side, dtype=torch.float64, device=DEV)
    pts = torch.stack(torch.meshgrid(ax, ax, indexing="ij"), -1).reshape(-1, 2)
    C = _sq_cost(pts, pts, torch.float32)
    rho = 2.0 / (2 * side * side)
    return [dict(C=C, p=_histogram(g, side).float(), q=_histogram(g, side).float(), rho=rho,
                 mu0=None, nu0=None) for _ in range(case["count"])]


def _network(case, seed):
    """Weights, inputs and targets of a training step of the warm start."""
    r = np.random.default_rng([6, int(seed)])
    dims = [case["inp"], case["hidden"], case["hidden"], case["out"]]
    flat = []
    for a, b in zip(dims, dims[1:]):
        lim = math.sqrt(6.0 / a)
        flat += [r.uniform(-lim, lim, a * b), r.uniform(-0.05, 0.05, b)]
    g = _gen(seed)
    x = -torch.log1p(-_rand(g, case["batch"], case["inp"]))  # histograms of mean 1
    t = torch.randn(case["batch"], case["out"], generator=g, device=DEV)
    return dims, np.concatenate(flat).astype(np.float32), x.float(), t


# ---------------------------------------------------------------------------
# The library's calls.
# ---------------------------------------------------------------------------
FLAGS = {"compensated": drot.FLAG_COMPENSATED, "skip_c": drot.FLAG_SKIP_C}
KIND = {"bf16": drot.COST_BF16, "coords": drot.COST_COORDS}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        dims, w, x, t = _network(case, seed)
        net = drot.MLP(dims[0], dims[1], dims[3], max_batch=case["batch"])
        net.set_weights(w)
        return dict(case=case, net=net, x=x, t=t)
    if kind == "solve":
        pr = _problem(case, seed)
        if "C" in pr and case.get("padded", True):
            pr["C"] = drot.padded(pr["C"])
        return dict(case=case, pr=pr)
    probs = _batch_problems(case, seed) if kind == "batch" else _grid_problems(case, seed)
    shared = {}
    for pr in probs:
        pr["C"] = shared.setdefault(pr["C"].data_ptr(), drot.padded(pr["C"]))
        pr["tol"] = 0.0
    return dict(case=case, probs=probs)


def run(state):
    case = state["case"]
    if case["kind"] == "mlp":
        if case["op"] == "forward":
            return state["net"].forward(state["x"])
        loss, grad = state["net"].gradients(state["x"], state["t"])
        return np.float32(loss), grad
    if case["kind"] == "solve":
        pr, cost = state["pr"], case["cost"]
        args = dict(tol=0.0, max_iter=case["iters"], mu0=pr["mu0"], nu0=pr["nu0"],
                    flags=FLAGS.get(case.get("option"), 0))
        if cost in KIND:
            X, res, mu, nu = drot.solve_cost(case["m"], case["n"], pr["p"], pr["q"], pr["rho"],
                                             KIND[cost], C=pr.get("C"), xs=pr.get("xs"),
                                             xt=pr.get("xt"), **args)
        else:
            X, res, mu, nu = drot.solve(pr["C"], pr["p"], pr["q"], pr["rho"], **args)
        if X.dtype == torch.float64:
            return X, mu, nu, res["objective"], res["iters"]
        return X, mu.float(), nu.float(), np.float32(res["objective"]), res["iters"]
    _, outs = drot.solve_batched(state["probs"], max_iter=case["iters"])
    if case["kind"] == "grid":
        return (torch.stack([mu for _, _, mu, _ in outs]).float(),
                torch.stack([nu for _, _, _, nu in outs]).float(),
                np.array([r["objective"] for _, r, _, _ in outs], dtype=np.float32))
    return [(X, mu.float(), nu.float()) for X, _, mu, nu in outs]


def _solve_work(m, n, iters, cost_bytes, size):
    # About nine operations per entry and iteration: the shift (two additions
    # and a product), the clamp, the row and column sums, <C, X> and the dual
    # residual.
    return dict(bytes=float(cost_bytes + size * (m * n + m + n) + 16 * (m + n)),
                flops=9.0 * m * n * iters)


def work(case):
    kind, iters = case["kind"], case.get("iters")
    if kind == "mlp":
        i, h, o, b = case["inp"], case["hidden"], case["out"], case["batch"]
        weights = i * h + h * h + h * o
        if case["op"] == "forward":
            return dict(bytes=4.0 * (weights + b * (i + o)), flops=2.0 * b * weights)
        return dict(bytes=4.0 * (2 * weights + b * (i + o)),
                    flops=2.0 * b * (3 * weights - i * h))
    if kind == "solve":
        m, n, cost = case["m"], case["n"], case["cost"]
        size = 8 if cost == "f64" else 4
        cb = {"bf16": 2 * m * n, "coords": 4 * case.get("dim", 2) * (m + n)}.get(cost, size * m * n)
        return _solve_work(m, n, iters, cb, size)
    if kind == "grid":
        N, count = case["side"] ** 2, case["count"]
        one = _solve_work(N, N, iters, 0, 4)
        return dict(bytes=4.0 * N * N + count * one["bytes"], flops=count * one["flops"])
    mean = (case["lo"] + case["hi"]) / 2
    one = _solve_work(mean, mean, iters, 4 * mean * mean, 4)
    return dict(bytes=case["count"] * one["bytes"], flops=case["count"] * one["flops"])


# ---------------------------------------------------------------------------
# The same in plain 64-bit torch.
# ---------------------------------------------------------------------------
def _iterate(C, p, q, rho, iters, mu0=None, nu0=None):
    """Algorithm 1 of the paper in float64: X_K, mu_K, nu_K and <C, X_K>."""
    p, q = p.double(), q.double()
    m, n = p.numel(), q.numel()
    rC = rho * C
    phi = torch.zeros_like(p) if mu0 is None else rho * mu0
    psi = torch.zeros_like(q) if nu0 is None else rho * nu0
    X = torch.outer(p, q)
    a = X.sum(1) - p + n * phi + psi.sum()
    b = X.sum(0) - q + m * psi + phi.sum()
    alpha = a.sum() / (m + n)
    for _ in range(iters):
        X += phi[:, None]
        X += psi
        X -= rC
        X.clamp_(min=0.0)
        r, s = X.sum(1) - p, X.sum(0) - q
        beta = r.sum() / (m + n)
        phi = (a - 2 * r + 2 * beta - alpha) / n
        psi = (b - 2 * s + 2 * beta - alpha) / m
        a, b, alpha = a - r, b - s, alpha - beta
    return X, phi / rho, psi / rho, float((C * X).sum())


def _exact_cost(pr):
    if "C" in pr:
        return pr["C"].double()
    xs, xt = pr["xs"].double(), pr["xt"].double()
    return _sq_cost(xs, xt, torch.float64)


def _exact_network(case, seed):
    dims, flat, x, t = _network(case, seed)
    x, t = x.double(), t.double()
    W, o = [], 0
    flat = torch.tensor(flat, device=DEV, dtype=torch.float64)
    for a, b in zip(dims, dims[1:]):
        W.append((flat[o:o + a * b].reshape(b, a), flat[o + a * b:o + a * b + b]))
        o += a * b + b
    acts = [x]
    for k, (w, b) in enumerate(W):
        z = acts[-1] @ w.t() + b
        acts.append(z.clamp(min=0.0) if k < 2 else z)
    if case["op"] == "forward":
        return acts[-1]
    diff = acts[-1] - t
    d, grads = 2 * diff / diff.numel(), []
    for k in (2, 1, 0):
        grads = [(d.t() @ acts[k]).flatten(), d.sum(0)] + grads
        if k:
            d = (d @ W[k][0]) * (acts[k] > 0)
    return float((diff ** 2).mean()), torch.cat(grads)


def exact(case, seed):
    if case["kind"] == "mlp":
        return _exact_network(case, seed)
    if case["kind"] == "solve":
        pr = _problem(case, seed)
        out = _iterate(_exact_cost(pr), pr["p"], pr["q"], pr["rho"], case["iters"], pr["mu0"],
                       pr["nu0"])
        return out + (None,)
    make = _batch_problems if case["kind"] == "batch" else _grid_problems
    outs = [_iterate(pr["C"].double(), pr["p"], pr["q"], pr["rho"], case["iters"])
            for pr in make(case, seed)]
    if case["kind"] == "grid":
        return (torch.stack([o[1] for o in outs]), torch.stack([o[2] for o in outs]),
                np.array([o[3] for o in outs]))
    return [o[:3] for o in outs]
