"""The one-workgroup iteration: shapes at the edges of its wave and lane
distribution against the oracle (tolerances of tests/test_gpu_parity.py), and
stops by tolerance, which come one iteration late and are made good by
repeating iterations from the last saved state: the result is bit for bit that
of a run with that many iterations."""
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


def _solve(ctx, inst, dtype, **kw):
    import torch
    from paper_2110_11738_amd import drot
    t = lambda a: torch.tensor(a, dtype=getattr(torch, dtype), device="cuda")
    X, res, mu, nu = drot.solve(t(inst.C), t(inst.p), t(inst.q), inst.rho, ctx=ctx, **kw)
    torch.cuda.synchronize()
    assert res["path"] == 1
    return res, [a.cpu().numpy() for a in (X, mu, nu)]


def _instance(m, n, dtype):
    inst = config_mixture_2d(41, m, n)
    return round_to(inst, np.float32) if dtype == "float32" else inst


@pytest.mark.parametrize("dtype,m,n", [
    ("float32", 11, 64), ("float32", 12, 65), ("float32", 176, 33), ("float32", 177, 64),
    ("float32", 255, 127), ("float32", 128, 255), ("float32", 63, 511), ("float32", 511, 2),
    ("float64", 11, 64), ("float64", 177, 63), ("float64", 127, 127), ("float64", 63, 200),
    ("float64", 31, 500)])
def test_trajectory(ctx, dtype, m, n):
    inst = _instance(m, n, dtype)
    K = 12
    print(f"[small] {dtype} {m}x{n}", flush=True)
    res, got = _solve(ctx, inst, dtype, tol=0.0, max_iter=K)
    tr = ctx.trace(1, K)
    R = ref.solve(inst.C, inst.p, inst.q, inst.rho, 0.0, max_iter=K, trace=True)
    assert res["iters"] == K and res["status"] == 1
    for g, r, tol in zip(got, (R.X, R.mu, R.nu), (TOL[dtype][0], TOL[dtype][1], TOL[dtype][1])):
        assert float(np.abs(g - r).max() / np.abs(r).max()) <= tol
    for c in range(5):
        scale = np.abs(R.trace[:, c]).max()
        assert float(np.abs(tr[:, c] - R.trace[:, c]).max()) <= (1e-9 if dtype == "float64" else 1e-3) * scale


@pytest.mark.parametrize("dtype,m,n", [("float32", 50, 60), ("float64", 23, 130)])
def test_stop_inside_a_launch(ctx, dtype, m, n):
    inst = _instance(m, n, dtype)
    K = 300
    _solve(ctx, inst, dtype, tol=0.0, max_iter=K)
    test = ctx.trace(1, K)[:, 5]
    low = [k for k in range(K) if k == 0 or test[k] < test[:k].min()]  # a tolerance stops there
    picks = sorted({low[0], low[-1]} | {low[i] for i in range(0, len(low), max(1, len(low) // 8))} |
                   {k for k in low if (k + 1) % 64 in (0, 1, 63)})
    for k in picks:
        a, x = _solve(ctx, inst, dtype, tol=float(test[k]), max_iter=K)
        b, y = _solve(ctx, inst, dtype, tol=0.0, max_iter=k + 1)
        print(f"[small] stop at {k + 1}: {a['iters']} {a['status']}", flush=True)
        assert (a["iters"], a["status"]) == (k + 1, 0) and b["iters"] == k + 1
        for u, v in zip(x, y):
            np.testing.assert_array_equal(u, v)
