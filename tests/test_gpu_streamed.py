"""Sweeps over problems beyond the last-level cache: each default tile (one or
two chunks per lane, two or four row blocks per workgroup) in each cost kind,
with whole and ragged widths.  The row blocks kept in the cache change how
memory is accessed and nothing else, so the result is bit-equal to the one
with streaming accesses throughout; both match the oracle (tolerances of
tests/test_gpu_parity.py: float32 chains are at most 16 entries long here)."""
import numpy as np
import pytest

from gen import dirichlet1
from oracle import ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2110_11738_amd import drot
    c = drot.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("kind,m,n", [
    ("float32", 5200, 5100), ("float32", 5201, 5103), ("float32", 27000, 1000),
    ("float32", 11700, 10800), ("float64", 3500, 3700), ("float64", 3501, 3701),
    ("coords", 7600, 6700), ("coords", 7601, 6701), ("bf16", 6000, 6104), ("bf16", 6001, 6105)])
def test_kept_blocks_and_tiles(ctx, kind, m, n):
    import torch
    from paper_2110_11738_amd import drot
    rng = np.random.default_rng([23, m, n])
    dt = torch.float64 if kind == "float64" else torch.float32
    npd = np.float64 if kind == "float64" else np.float32
    xs, xt = (rng.uniform(0, 1, (k, 2)).astype(np.float32) for k in (m, n))
    D = sum((xs[:, None, d].astype(np.float64) - xt[None, :, d]) ** 2 for d in range(2))
    D /= D.max()
    p, q = (dirichlet1(rng, k).astype(npd).astype(np.float64) for k in (m, n))
    src = {}
    if kind == "coords":
        code, src = drot.COST_COORDS, dict(xs=torch.tensor(xs, device="cuda"),
                                           xt=torch.tensor(xt, device="cuda"))
    else:
        code = drot.COST_BF16 if kind == "bf16" else drot.COST_DENSE
        C = torch.tensor(D).to(torch.bfloat16 if kind == "bf16" else dt)
        D = C.double().numpy()
        src = dict(C=drot.padded(C.cuda()))
    rho, K = 1.0 / np.log(m) / (m + n), 3
    pd, qd = (torch.tensor(a, dtype=dt, device="cuda") for a in (p, q))
    got = []
    for mode in (drot.CACHE_AUTO, drot.CACHE_STREAM):
        print(f"[streamed] {kind} {m}x{n} cache_mode {mode}", flush=True)
        X, res, mu, nu = drot.solve_cost(m, n, pd, qd, rho, code, tol=0.0, max_iter=K,
                                         cache_mode=mode, ctx=ctx, **src)
        torch.cuda.synchronize()
        assert res["iters"] == K and res["path"] == 0
        got.append((X.cpu().numpy(), mu.cpu().numpy(), nu.cpu().numpy()))
        del X
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    R = ref.solve(D, p, q, rho, 0.0, max_iter=K)
    tol = 1e-10 if kind == "float64" else 2e-5
    for a, b in zip(got[0], (R.X, R.mu, R.nu)):
        assert float(np.abs(a - b).max() / np.abs(b).max()) <= tol
