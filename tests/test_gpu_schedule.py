"""Schedules of the register-phase launches: grids below what the machine holds
(spread over the CUs), items that do not divide an instance's tiles, fewer
workgroups per CU than fit, and the work queue launch after launch, against
the C oracle."""
import numpy as np
import pytest

import games
import oracle
from helpers import normwise, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-6)])
@pytest.mark.parametrize("n,d,l", [(256, 11, 4), (260, 11, 1), (500, 14, 3), (516, 12, 2),
                                   (772, 11, 2), (1000, 13, 2), (200, 15, 2), (100, 16, 4),
                                   (24, 18, 3), (1, 18, 3)])
def test_batches(n, d, l, dtype, tol):
    from paper_2601_01903_amd import BatchPlan
    say(f"[case] schedule {n} x d={d} l={l} {dtype}")
    np_t = np.float64 if dtype == "f64" else np.float32
    k = min(n, 4)
    v = [games.tree_values(games.tree_game(d, 30, 5, games.rng_for(973, d * 8 + i))).astype(np_t)
         for i in range(k)]
    x = torch.from_numpy(np.concatenate(v)).to(DEV).repeat(n // k).contiguous()
    bp = BatchPlan([d] * n, [l] * n, dtype=dtype)
    out = bp.apply(x, graph=False)
    m = bp.out_offset[1]
    rows = out.view(n, m)
    for i in range(k):
        ref = oracle.fsi_c(v[i].astype(np.float64), d, l, nthreads=16)
        assert normwise(rows[i].double().cpu().numpy(), ref) < tol
    assert torch.equal(rows, rows[:k].repeat(n // k, 1))
    for _ in range(3):
        got = torch.full_like(out, float("nan"))
        bp.apply(x * 2, out=got, graph=False)
        assert torch.equal(got, out * 2)
        bp.apply(x, out=got)
        assert torch.equal(got, out)
    bp.close()


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-6)])
def test_several_orders(dtype, tol):
    from paper_2601_01903_amd import BatchPlan
    say(f"[case] schedule of several orders {dtype}")
    np_t = np.float64 if dtype == "f64" else np.float32
    ds = [11 + i % 6 for i in range(330)]
    ls = [1 + i % 4 for i in range(330)]
    games_of = {d: games.tree_values(games.tree_game(d, 30, 5, games.rng_for(974, d))).astype(np_t)
                for d in set(ds)}
    x = torch.from_numpy(np.concatenate([games_of[d] for d in ds])).to(DEV)
    refs = {(d, l): oracle.fsi_c(games_of[d].astype(np.float64), d, l, nthreads=16)
            for d, l in set(zip(ds, ls))}
    bp = BatchPlan(ds, ls, dtype=dtype)
    out = bp.apply(x, graph=False)
    o = out.double().cpu().numpy()
    for i, (d, l) in enumerate(zip(ds, ls)):
        assert normwise(o[bp.out_offset[i]:bp.out_offset[i + 1]], refs[d, l]) < tol, (i, d, l)
    assert torch.equal(bp.apply(x), out)
    bp.close()
