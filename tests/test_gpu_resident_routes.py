"""Which launches the iterations of a problem that fits the chip run as, and that
the ways off the chip give the same result: launches called off because their
workgroups are not all there, streams with fewer compute units.  Within a path, splitting the iterations into calls
changes no bit.  The library counts its launches and lets a test
force such conditions (drot_internal_counts and drot_internal_rare)."""
import ctypes

import numpy as np
import pytest

from gen import config_mixture_2d, round_to

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx():
    from paper_2110_11738_amd import drot
    c = drot.Context(0)
    yield c
    c.close()


def _counts(ctx):
    """Resident launches, graph replays, iterations launched singly."""
    return _all_counts(ctx)[:3]


def _all_counts(ctx):
    """The same, and iterations of the bound problem repeated after a stop."""
    from paper_2110_11738_amd import drot
    out = (ctypes.c_int64 * 4)()
    drot.lib().drot_internal_counts(ctx.handle, out)
    return np.array(out)


def _rare(ctx, gate_polls=1 << 20, refuse_after=-1):
    from paper_2110_11738_amd import drot
    drot.lib().drot_internal_rare(ctx.handle, ctypes.c_int(gate_polls),
                                  ctypes.c_int64(refuse_after))


def _problem(m, n, dtype, seed=51):
    import torch
    inst = config_mixture_2d(seed, m, n)
    if dtype == "float32":
        inst = round_to(inst, np.float32)
    t = lambda a: torch.tensor(a, dtype=getattr(torch, dtype), device="cuda")
    return t(inst.C), t(inst.p), t(inst.q), inst.rho


def _steps(ctx, prob, calls, **kw):
    """bind, calls of iterate, finish: plan, duals and trace (without times)."""
    import torch
    from paper_2110_11738_amd import drot
    C, p, q, rho = prob
    X = torch.empty_like(C)
    mu, nu = (torch.empty(k, dtype=torch.float64, device="cuda") for k in C.shape)
    ctx.bind(C, p, q, X, drot.make_params(rho, 0.0, 10 ** 6, **kw))
    for k in calls:
        ctx.iterate(k)
    res = ctx.finish(mu, nu)
    assert res["iters"] == sum(calls)
    return X, mu, nu, torch.tensor(ctx.trace(1, sum(calls))[:, [0, 1, 2, 3, 4, 5, 7]])


def _same(a, b):
    import torch
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,m,n", [("float32", 700, 300), ("float64", 1100, 260)])
def test_called_off_launches_are_made_up_by_sweeps(ctx, dtype, m, n):
    prob = _problem(m, n, dtype)
    on_chip = _steps(ctx, prob, (40, 24))
    _rare(ctx, refuse_after=0)
    c0 = _counts(ctx)
    sweeps = _steps(ctx, prob, (40, 24))
    assert _counts(ctx)[0] == c0[0]
    _rare(ctx, gate_polls=0)
    c0 = _counts(ctx)
    _same(_steps(ctx, prob, (40, 24)), sweeps)
    assert _counts(ctx)[0] == c0[0] + 2  # both went out, and gave up
    _rare(ctx)
    c0 = _counts(ctx)
    _same(_steps(ctx, prob, (40, 24)), on_chip)  # nothing is left behind
    assert tuple(_counts(ctx) - c0) == (2, 0, 0)


def test_called_off_launches_of_a_solve_a_checkpoint_and_a_batch(ctx):
    import torch
    from paper_2110_11738_amd import drot
    prob = _problem(300, 700, "float64")
    C, p, q, rho = prob

    def runs():
        X, res, mu, nu = drot.solve(C, p, q, rho, tol=2e-2, max_iter=5000, ctx=ctx)
        assert res["status"] == 0
        Xc = torch.empty_like(C)
        ctx.bind(C, p, q, Xc, drot.make_params(rho, 0.0, 100))
        ctx.iterate(50)
        blob = ctx.checkpoint()
        Xs = Xc.clone()
        ctx.bind(C, p, q, Xs, drot.make_params(rho, 0.0, 100, x0_mode=drot.X0_GIVEN))
        ctx.resume(blob)
        ctx.iterate(50)
        assert ctx.finish()["iters"] == 100
        return X, mu, nu, Xs

    def batch():
        probs = [dict(C=C[:k].contiguous(), p=p[:k] / p[:k].sum(), q=q, rho=rho, tol=0.0)
                 for k in (300, 40, 150)]
        for pr in probs:
            pr["q"] = pr["q"] * (pr["p"].sum() / pr["q"].sum())
        rc, outs = drot.solve_batched(probs, max_iter=60, ctx=ctx)
        assert rc == drot.MAXITER and all(r["iters"] == 60 for _, r, _, _ in outs)
        return [t for X, _, mu, nu in outs for t in (X, mu, nu)]

    _rare(ctx, refuse_after=0)
    sweeps, one_by_one = runs(), batch()
    _rare(ctx, gate_polls=0)
    c0 = _counts(ctx)
    _same(runs(), sweeps)
    # a team of one workgroup has nobody to wait for
    off = batch()
    assert _counts(ctx)[0] > c0[0] + 2
    for a, b in zip(off, one_by_one):
        assert float((a - b).abs().max()) <= 1e-10 * float(b.abs().max())


@pytest.mark.parametrize("dtype,m,n", [("float32", 700, 300), ("float32", 1300, 2700),
                                       ("float64", 1100, 260)])
def test_splitting_calls_changes_no_bit(ctx, dtype, m, n):
    """40 iterations in one call and in several, with single iterations among
    them, with a checkpoint after any of them, and a solve of 1030 (1024 and 6)."""
    import torch
    from paper_2110_11738_amd import drot
    prob = _problem(m, n, dtype)
    C, p, q, rho = prob
    whole = _steps(ctx, prob, (40,))
    for calls in ((37, 3), (1, 39), (7, 1, 31, 1)):
        _same(_steps(ctx, prob, calls), whole)
    prm = dict(rho=rho, tol=0.0, max_iter=100)
    X = torch.empty_like(C)
    ctx.bind(C, p, q, X, drot.make_params(**prm))
    ctx.iterate(37)
    blob = ctx.checkpoint()
    other = drot.Context(0)
    try:
        Y = X.clone()
        other.bind(C, p, q, Y, drot.make_params(x0_mode=drot.X0_GIVEN, **prm))
        other.resume(blob)
        other.iterate(3)
        assert other.finish()["iters"] == 40
        assert torch.equal(Y, whole[0])
    finally:
        other.close()
    X, res, mu, nu = drot.solve(C, p, q, rho, tol=0.0, max_iter=1030, ctx=ctx)
    assert res["iters"] == 1030
    _same((X, mu, nu), _steps(ctx, prob, (500, 530))[:3])


def _few_units():
    """A stream on half of the compute units."""
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    units = torch.cuda.get_device_properties(0).multi_processor_count
    words = (units + 31) // 32
    mask = (ctypes.c_uint32 * words)(*([0xffffffff] * (words // 2)))
    s = ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(s), ctypes.c_uint32(words), mask) == 0
    return torch.cuda.ExternalStream(s.value), lambda: hip.hipStreamDestroy(s)


def test_a_stream_with_fewer_units_replays_graphs(ctx):
    """The sweeps of a problem that would fit the chip go out as on any other
    stream: graphs of 32 iterations, and no more than that after a stop."""
    import torch
    from paper_2110_11738_amd import drot
    C, p, q, rho = _problem(2100, 2500, "float32")  # more tiles than half of the units
    _rare(ctx, refuse_after=0)
    a = drot.solve(C, p, q, rho, tol=0.0, max_iter=100, ctx=ctx)
    tol = float(ctx.trace(1, 100)[:, 5].min()) * 1.0000001
    at = int(np.argmax(ctx.trace(1, 100)[:, 5] <= tol)) + 1
    _rare(ctx)
    s, drop = _few_units()
    torch.cuda.synchronize()
    c0 = _counts(ctx)
    b = drot.solve(C, p, q, rho, tol=0.0, max_iter=100, ctx=ctx, stream=s)
    assert tuple(_counts(ctx) - c0) == (0, 3, 4)
    _same((a[0], a[2], a[3]), (b[0], b[2], b[3]))
    c0 = _counts(ctx)
    d = drot.solve(C, p, q, rho, tol=tol, max_iter=2000, ctx=ctx, stream=s)
    assert d[1]["iters"] == at and d[1]["status"] == 0
    assert tuple(_counts(ctx) - c0) == (0, (at + 31) // 32, 0)
    torch.cuda.synchronize()
    drop()


@pytest.mark.parametrize("m,n", [(100, 90), (300, 700)])
@pytest.mark.parametrize("rho,cost", [(1e-50, 1.0), (1e-12, 1e-30), (1e25, 1e20)])
def test_products_beyond_the_element_type_take_sweeps(ctx, m, n, rho, cost):
    """rho times the cost is below float32's normal numbers, or beyond its range:
    alone, and in a batch beside an ordinary problem."""
    from paper_2110_11738_amd import drot
    C, p, q, _ = _problem(m, n, "float32")
    C = C * cost
    X, res, mu, nu = drot.solve(C, p, q, rho, tol=0.0, max_iter=20, ctx=ctx)
    tr = ctx.trace(1, 20)
    assert res["iters"] == 20 and np.isfinite(tr).all()
    # <C, X> of the last iteration: float32 sums of at most 512 entries
    assert abs(tr[19, 0] - res["objective"]) <= 1e-6 * abs(res["objective"])
    c0 = _counts(ctx)
    rc, outs = drot.solve_batched([dict(C=C, p=p, q=q, rho=rho, tol=0.0),
                                   dict(C=_problem(m, n, "float32")[0], p=p, q=q, rho=1e-3, tol=0.0)],
                                  max_iter=20, ctx=ctx)
    assert rc == drot.MAXITER and all(r["iters"] == 20 for _, r, _, _ in outs)
    assert _counts(ctx)[0] - c0[0] == 1


@pytest.mark.parametrize("dtype,m,n", [("float32", 4000, 4000), ("float32", 4001, 4001),
                                       ("float32", 3999, 4003), ("float64", 4000, 2047),
                                       ("float32", 3300, 3203)])
def test_a_stop_repeats_no_more_than_since_a_saved_state(ctx, dtype, m, n):
    """Whole and ragged widths, aligned rows and not, up to the tallest tiles: a
    stop beyond 300 iterations repeats at most 256 and the two the test trails by."""
    from paper_2110_11738_amd import drot
    C, p, q, rho = _problem(m, n, dtype)
    K = 700
    X, res, mu, nu = drot.solve(C, p, q, rho, tol=0.0, max_iter=K, ctx=ctx)
    test = ctx.trace(1, K)[:, 5]
    at = max(k for k in range(K) if k == 0 or test[k] < test[:k].min())
    assert at > 300
    c0 = _counts(ctx)
    Y, res, mu2, nu2 = drot.solve(C, p, q, rho, tol=float(test[at]), max_iter=2000, ctx=ctx)
    assert (res["iters"], res["status"]) == (at + 1, 0)
    assert tuple(_counts(ctx) - c0) == (1, 0, 0)
    print(f"[saved] {dtype} {m}x{n} stop at {at + 1}, {_all_counts(ctx)[3]} repeated", flush=True)
    assert _all_counts(ctx)[3] <= 258
    Z, res, mu, nu = drot.solve(C, p, q, rho, tol=0.0, max_iter=at + 1, ctx=ctx)
    _same((Y, mu2, nu2), (Z, mu, nu))


@pytest.mark.parametrize("dtype,m,n", [
    ("float32", 129, 129), ("float32", 32, 1025), ("float32", 1024, 255), ("float32", 1025, 257),
    ("float32", 2080, 3840), ("float32", 4095, 4096), ("float32", 16500, 9), ("float32", 4096, 5),
    ("float32", 12, 16640), ("float64", 65, 257), ("float64", 1100, 1030), ("float64", 2100, 2561),
    ("float64", 4000, 2047), ("float64", 600, 26)])
def test_shapes_that_run_on_the_chip(ctx, dtype, m, n):
    """The shapes whose results tests/test_gpu_resident.py compares with the oracle."""
    import torch
    from paper_2110_11738_amd import drot
    dt = getattr(torch, dtype)
    p, q = (torch.full((k,), 1.0 / 32768, dtype=dt, device="cuda") for k in (m, n))
    p[0] += 1 - p.double().sum().item()
    q[0] += 1 - q.double().sum().item()
    drot.solve(torch.rand(m, n, dtype=dt, device="cuda"), p, q, 1.0 / (m + n), tol=0.0, max_iter=12,
               ctx=ctx)
    assert tuple(_counts(ctx)) == (1, 0, 0)


def test_a_captured_call_is_sweeps(ctx):
    """iterate() into a capture, replayed between other work, then on-chip calls."""
    import torch
    from paper_2110_11738_amd import drot
    C, p, q, rho = _problem(300, 700, "float64")

    def run(capture):
        X = torch.empty_like(C)
        ctx.bind(C, p, q, X, drot.make_params(rho, 0.0, 1000))
        states = []
        if capture:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                ctx.iterate(40, stream=torch.cuda.current_stream())
        for _ in range(3):
            if capture:
                g.replay()
            else:
                ctx.iterate(40)
            torch.cuda.synchronize()
            states.append(X.clone())
            _ = torch.rand(1000, 1000, device="cuda") @ torch.rand(1000, 1000, device="cuda")
        c0 = _counts(ctx)
        if capture:
            assert ctx.poll()[0] == 120
            ctx.iterate(20)
            assert tuple(_counts(ctx) - c0) == (1, 0, 0)
            assert ctx.finish()["iters"] == 140
        return states

    _rare(ctx, refuse_after=0)
    sweeps = run(False)
    _rare(ctx)
    c0 = _counts(ctx)
    replayed = run(True)
    assert tuple(_counts(ctx) - c0) == (1, 0, 40)  # recorded once
    _same(replayed, sweeps)


def test_two_threads_with_a_context_and_a_stream_each():
    import threading
    import torch
    from paper_2110_11738_amd import drot
    probs = [_problem(700, 300, "float32", 61), _problem(1300, 900, "float32", 62)]
    want, got, errors = [None, None], [[], []], []
    ctxs = [drot.Context(0), drot.Context(0)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]

    def solve(k):
        C, p, q, rho = probs[k]
        X, res, mu, nu = drot.solve(C, p, q, rho, tol=0.0, max_iter=300, ctx=ctxs[k])
        assert res["iters"] == 300
        torch.cuda.current_stream().synchronize()
        return X, mu, nu

    for k in range(2):
        want[k] = solve(k)
    torch.cuda.synchronize()

    def work(k):
        try:
            with torch.cuda.stream(streams[k]):
                for _ in range(5):
                    got[k].append(solve(k))
        except Exception as e:
            errors.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    for k in range(2):
        assert _counts(ctxs[k])[0] == 6
        for out in got[k]:
            _same(out, want[k])
        ctxs[k].close()


def test_a_batch_whose_second_launch_is_refused(ctx):
    """The launches before it have run; the sweeps take every problem on from
    where it stands."""
    from paper_2110_11738_amd import drot
    probs = []
    for k in range(12):
        C, p, q, rho = _problem(1500, 1400, "float64", 70 + k)
        probs.append(dict(C=C, p=p, q=q, rho=rho, tol=0.0))
    rc, want = drot.solve_batched(probs, max_iter=50, ctx=ctx)
    launches = _counts(ctx)[0]
    assert launches > 1
    _rare(ctx, refuse_after=1)
    rc, outs = drot.solve_batched(probs, max_iter=50, ctx=ctx)
    assert rc == drot.MAXITER and _counts(ctx)[0] == launches + 1
    for (X, res, mu, nu), (X0, _, mu0, nu0) in zip(outs, want):
        assert res["iters"] == 50
        for a, b in ((X, X0), (mu, mu0), (nu, nu0)):  # float64: sums in another order
            assert float((a - b).abs().max()) <= 1e-10 * float(b.abs().max())


def test_batch_tuner_times_what_the_solver_runs(ctx):
    """Problems on the chip have no schedule to choose: the tuner times their
    launches, leaves the cache alone and tunes the others."""
    from paper_2110_11738_amd import drot
    fit = [dict(zip("Cpq", _problem(k, 700, "float32", 80)[:3]), rho=1e-3, tol=0.0)
           for k in (300, 600, 900)]
    table = drot.tune_batched(fit, iters=64, ctx=ctx)
    launches, _, _ = _counts(ctx)
    assert launches == 2  # one to warm up, one timed
    assert sum(t["problems"] for t in table) == 3
    for t in table:  # untuned
        assert (t["tile_rows"], t["blocks_per_item"], t["chunks"]) == (16, 1, 2)
        assert t["us_per_iter"] > 0
    drot.tune_batched(fit, iters=64, check_every=16, ctx=ctx)  # swept
    assert _counts(ctx)[0] == launches
    big = dict(zip("Cpq", _problem(4500, 4400, "float32", 81)[:3]), rho=1e-4, tol=0.0)
    table = drot.tune_batched(fit + [big], iters=32, ctx=ctx)
    assert _counts(ctx)[0] == launches + 2
    assert sum(t["problems"] for t in table) == 4
    t = [t for t in table if (t["m_class"], t["n_class"]) == (5, 5)][0]
    assert t["tile_rows"] in (8, 16, 32) and t["blocks_per_item"] in (1, 2, 4) and t["chunks"] in (1, 2)
    rc, outs = drot.solve_batched(fit + [big], max_iter=40, ctx=ctx)
    assert rc == drot.MAXITER and all(r["iters"] == 40 for _, r, _, _ in outs)
    bad = dict(fit[2], p=fit[2]["p"] * 2)
    with pytest.raises(drot.DrotError, match="problem 2:"):
        drot.tune_batched([big, fit[0], bad], iters=32, ctx=ctx)


def test_tuning_over_few_iterations_times_the_bound_path(ctx):
    import torch
    from paper_2110_11738_amd import drot
    C, p, q, rho = _problem(300, 700, "float32")
    ctx.bind(C, p, q, torch.empty_like(C), drot.make_params(rho, 0.0, 1000))
    for iters in (1, 3, 20):
        c0 = _counts(ctx)
        best, us = ctx.tune(iters)
        assert tuple(_counts(ctx) - c0) == (2, 0, 0) and us > 0
        c0 = _counts(ctx)
        table = drot.tune_batched([dict(C=C, p=p, q=q, rho=rho, tol=0.0)], iters=iters, ctx=ctx)
        assert tuple(_counts(ctx) - c0) == (2, 0, 0) and table[0]["us_per_iter"] > 0
        ctx.bind(C, p, q, torch.empty_like(C), drot.make_params(rho, 0.0, 1000))


FIRST = """
import time, torch
from paper_2110_11738_amd import drot
ctx = drot.Context(0)
C = torch.rand(517, 483, device="cuda")
p, q = (torch.full((k,), 1.0 / 8192, device="cuda") for k in C.shape)
p[0] += 1 - p.double().sum().item()
q[0] += 1 - q.double().sum().item()
ctx.bind(C, p, q, torch.empty_like(C), drot.make_params(1e-3, 0.0, 1000))
torch.cuda.synchronize()
for _ in range(3):
    t = time.perf_counter()
    ctx.iterate(20)
    torch.cuda.synchronize()
    print("took", time.perf_counter() - t, flush=True)
"""


def test_the_first_iterations_of_a_process_take_no_longer():
    """What a process's first cooperative launch sets up (17 ms) is there with the
    context."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", FIRST], cwd=root, capture_output=True, text=True,
                         timeout=90)
    assert out.returncode == 0, out.stderr
    first, second, third = (float(l.split()[1]) for l in out.stdout.splitlines() if l.startswith("took"))
    print(f"[first] {1e6 * first:.0f} us, then {1e6 * second:.0f} and {1e6 * third:.0f}", flush=True)
    assert first < third + 5e-3
