"""The resident iteration (plan and cost on the chip, tiles exchanging their
sums through memory) against the oracle: one shape for each tile height and
type, at the edges of tiles; stops inside a launch; launches mixed with single
iterations, which run as sweep + aux.

Tolerances are those of tests/test_gpu_parity.py: in float64 only the order of
the sums differs; in float32 a lane's sums run over at most 8 entries, a row's
over 4 entries and 6 levels, and everything after that is float64, so the
bound derived there for longer chains holds."""
import numpy as np
import pytest

from gen import config_mixture_2d, round_to
from oracle import ref

pytestmark = pytest.mark.gpu

TOL = {"float64": (1e-10, 1e-9), "float32": (2e-5, 2e-5)}


@pytest.fixture(scope="module")
def ctx():
    from paper_2110_11738_amd import drot
    c = drot.Context(0)
    yield c
    c.close()


def _inputs(inst, dtype):
    import torch
    t = lambda a: torch.tensor(a, dtype=getattr(torch, dtype), device="cuda")
    return t(inst.C), t(inst.p), t(inst.q)


def _instance(seed, m, n, dtype):
    inst = config_mixture_2d(seed, m, n)
    return round_to(inst, np.float32) if dtype == "float32" else inst


def _rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


# Tiles are 8 h rows by 256 (float32) or 128 (float64) columns, h = 4 up to 32
# tile rows, then 8, 16, 24, 32 as far as 256 tiles hold the problem.
@pytest.mark.parametrize("dtype,m,n", [
    ("float32", 129, 129), ("float32", 32, 1025), ("float32", 33, 513), ("float32", 1024, 255),
    ("float32", 1025, 257), ("float32", 2048, 2049), ("float32", 2080, 3840),
    ("float32", 4095, 4096), ("float32", 16500, 9),
    ("float64", 65, 257), ("float64", 1024, 127), ("float64", 1100, 1030),
    ("float64", 2049, 1024), ("float64", 2100, 2561), ("float64", 4000, 2047)])
def test_trajectory(ctx, dtype, m, n):
    import torch
    from paper_2110_11738_amd import drot
    inst = _instance(31, m, n, dtype)
    K = 12
    print(f"[resident] {dtype} {m}x{n}", flush=True)
    X, res, mu, nu = drot.solve(*_inputs(inst, dtype), inst.rho, tol=0.0, max_iter=K, ctx=ctx)
    torch.cuda.synchronize()
    tr = ctx.trace(1, K)
    R = ref.solve(inst.C, inst.p, inst.q, inst.rho, 0.0, max_iter=K, trace=True)
    assert res["iters"] == K and res["status"] == 1 and res["path"] == 0
    assert _rel(X.double().cpu().numpy(), R.X) <= TOL[dtype][0]
    assert _rel(mu.cpu().numpy(), R.mu) <= TOL[dtype][1]
    assert _rel(nu.cpu().numpy(), R.nu) <= TOL[dtype][1]
    np.testing.assert_array_equal(tr[:, 7], np.arange(1, K + 1))
    for c in range(5):  # pobj, dobj, r_primal, lagged r_dual, gap
        assert _rel(tr[:, c], R.trace[:, c]) <= (1e-9 if dtype == "float64" else 1e-3)


@pytest.mark.parametrize("m,n,at", [(300, 260, 1), (300, 260, 2), (1100, 140, 3), (200, 333, 64),
                                    (64, 700, 1023), (64, 700, 1025)])
def test_stops_inside_a_launch(ctx, m, n, at):
    """A tolerance between the oracle's test values stops the run at exactly
    that iteration, with X, the duals and the trace of that iteration."""
    import torch
    from paper_2110_11738_amd import drot
    inst = _instance(32, m, n, "float64")
    R = ref.solve(inst.C, inst.p, inst.q, inst.rho, 0.0, max_iter=at + 5, trace=True)
    test = R.trace[:, 5]
    tol = 1.000001 * test[:at].min()
    at = int(np.argmax(test <= tol)) + 1
    R = ref.solve(inst.C, inst.p, inst.q, inst.rho, 0.0, max_iter=at, trace=True)
    X, res, mu, nu = drot.solve(*_inputs(inst, "float64"), inst.rho, tol=tol, max_iter=5000,
                                ctx=ctx)
    torch.cuda.synchronize()
    tr = ctx.trace(1, at)
    assert res["status"] == 0 and res["iters"] == at
    assert _rel(X.cpu().numpy(), R.X) <= TOL["float64"][0]
    assert _rel(mu.cpu().numpy(), R.mu) <= TOL["float64"][1]
    assert _rel(tr[:, 5], R.trace[:, 5]) <= 1e-9


@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_mixed_with_single_iterations_and_repeated(ctx, dtype):
    import torch
    from paper_2110_11738_amd import drot
    inst = _instance(33, 700, 300, dtype)
    C, p, q = _inputs(inst, dtype)
    X = torch.empty_like(C)
    plans = []
    for _ in range(2):
        ctx.bind(C, p, q, X, drot.make_params(inst.rho, 0.0, 100))
        for k in (20, 1, 8, 3, 9):
            ctx.iterate(k)
        mu = torch.empty(700, dtype=torch.float64, device="cuda")
        nu = torch.empty(300, dtype=torch.float64, device="cuda")
        res = ctx.finish(mu, nu)
        plans.append((X.clone(), mu.clone(), nu.clone()))
    R = ref.solve(inst.C, inst.p, inst.q, inst.rho, 0.0, max_iter=41)
    assert res["iters"] == 41
    assert _rel(plans[0][0].double().cpu().numpy(), R.X) <= TOL[dtype][0]
    assert _rel(plans[0][1].cpu().numpy(), R.mu) <= TOL[dtype][1]
    for a, b in zip(*plans):
        assert torch.equal(a, b)


SIDES = [(5, 3), (1, 37), (40, 70), (129, 300), (1, 1), (300, 129), (700, 900), (1030, 260),
         (257, 1300), (64, 2048), (2000, 40), (1500, 1400)]


@pytest.mark.parametrize("dtype,K,extra", [("float32", 40, []), ("float64", 33, []),
                                           ("float32", 9, [(4200, 4100)] + [(1024, 1024)] * 20)])
def test_batch_trajectories(ctx, dtype, K, extra):
    """Problems from 1 x 1 up side by side, some batches with more than one
    launch and with a problem that does not fit the chip."""
    import torch
    from paper_2110_11738_amd import drot
    insts = [_instance(40 + k, m, n, dtype) for k, (m, n) in enumerate(SIDES + extra)]
    probs = [dict(zip("Cpq", _inputs(i, dtype)), rho=i.rho, tol=0.0) for i in insts]
    for k in range(0, len(probs), 2):
        probs[k]["C"] = drot.padded(probs[k]["C"])
    rc, outs = drot.solve_batched(probs, max_iter=K, ctx=ctx)
    torch.cuda.synchronize()
    assert rc == drot.MAXITER
    for inst, (X, res, mu, nu) in zip(insts, outs):
        R = ref.solve(inst.C, inst.p, inst.q, inst.rho, 0.0, max_iter=K)
        assert res["iters"] == K
        assert _rel(X.double().cpu().numpy(), R.X) <= TOL[dtype][0]
        scale = max(np.abs(R.mu).max(), np.abs(R.nu).max())
        assert np.abs(mu.cpu().numpy() - R.mu).max() <= TOL[dtype][1] * scale
        assert np.abs(nu.cpu().numpy() - R.nu).max() <= TOL[dtype][1] * scale


def test_batch_stops_each_problem_on_its_own(ctx):
    import torch
    from paper_2110_11738_amd import drot
    insts = [_instance(60 + k, m, n, "float64")
             for k, (m, n) in enumerate([(60, 50), (200, 333), (300, 260), (90, 400)])]
    probs = [dict(zip("Cpq", _inputs(i, "float64")), rho=i.rho, tol=t)
             for i, t in zip(insts, (3e-2, 2e-2, 5e-2, 1e-2))]
    rc, outs = drot.solve_batched(probs, max_iter=20000, check_every=200, ctx=ctx)
    torch.cuda.synchronize()
    assert rc == drot.OK
    for inst, pr, (X, res, mu, nu) in zip(insts, probs, outs):
        R = ref.solve(inst.C, inst.p, inst.q, inst.rho, pr["tol"], max_iter=20000)
        assert res["status"] == 0 and res["iters"] == R.info["iters"]
        assert _rel(X.cpu().numpy(), R.X) <= TOL["float64"][0]


# Few columns or one tile row: the column sums that cross tiles unrounded.
@pytest.mark.parametrize("dtype,m,n", [
    ("float32", 257, 128), ("float32", 583, 26), ("float32", 4096, 5), ("float32", 32, 513),
    ("float32", 9, 530), ("float32", 12, 16640), ("float64", 32, 513), ("float64", 600, 26)])
def test_trajectory_few_rows_or_columns(ctx, dtype, m, n):
    test_trajectory(ctx, dtype, m, n)


# Stops on both sides of saved states (after 32 iterations beyond 32 tile rows,
# else 128; doubling; then every 256), against runs of that many iterations.
@pytest.mark.parametrize("dtype,m,n", [("float32", 300, 301), ("float32", 1100, 40),
                                       ("float64", 257, 300), ("float32", 3300, 3200),
                                       ("float32", 3300, 3203)])
def test_stop_after_saved_states(ctx, dtype, m, n):
    import torch
    from paper_2110_11738_amd import drot
    inst = _instance(43, m, n, dtype)
    args = _inputs(inst, dtype)
    K = 620

    def solve(tol, max_iter):
        X, res, mu, nu = drot.solve(*args, inst.rho, tol=tol, max_iter=max_iter, ctx=ctx)
        torch.cuda.synchronize()
        return res, (X, mu, nu)

    solve(0.0, K)
    test = ctx.trace(1, K)[:, 5]
    low = [k + 1 for k in range(K) if k == 0 or test[k] < test[:k].min()]  # a tolerance stops there
    picks = {low[0], low[-1]}
    for save in (32, 64, 128, 256, 512):
        picks |= {k for k in low if abs(k - save) <= 1}
        picks |= {max([k for k in low if k <= save + 40], default=low[0])}
    for k in sorted(picks):
        if k < 8:
            continue  # solve(0, k) would be single iterations, sweep + aux
        a, x = solve(float(test[k - 1]), K)
        b, y = solve(0.0, k)
        print(f"[resident] {m}x{n} stop at {k}: {a['iters']} {a['status']}", flush=True)
        assert (a["iters"], a["status"], a["path"]) == (k, 0, 0) and b["iters"] == k
        for u, v in zip(x, y):
            assert torch.equal(u, v)


@pytest.mark.parametrize("dtype,m,n", [("float32", 4000, 4000), ("float32", 4001, 4001),
                                       ("float32", 4000, 4003), ("float64", 4000, 2047)])
def test_stop_after_saved_states_in_the_tallest_tiles(ctx, dtype, m, n):
    """32 rows per wave: half of rho C in LDS, which a save may not touch and a
    repeat loads again."""
    test_stop_after_saved_states(ctx, dtype, m, n)
