"""Instances of one work item, whose scores the register-phase kernel writes
itself, and the first sizes past them (the reduction kernel), alone and side by
side in a batch, over repeated launches through every entry point."""
import numpy as np
import pytest

import games
import oracle
from helpers import normwise, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def values(d, seed):
    return games.tree_values(games.tree_game(d, 30, 5, games.rng_for(951, seed)))


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-6)])
@pytest.mark.parametrize("d", [3, 10, 11, 12, 13, 14, 15, 16])
def test_single(d, dtype, tol):
    from paper_2601_01903_amd import Plan
    for l in range(1, min(4, d) + 1):
        say(f"[case] fold single d={d} l={l} {dtype}")
        v = values(d, d).astype(np.float64 if dtype == "f64" else np.float32)
        ref = oracle.fsi_c(v.astype(np.float64), d, l, nthreads=8)
        plan = Plan(d, l, dtype=dtype)
        x = torch.from_numpy(v).to(DEV)
        for rep in range(3):
            out = plan.apply(x * (rep + 1))
            got = out.double().cpu().numpy() / (rep + 1)
            assert normwise(got, ref) < tol, (l, rep)
        plan.close()


def test_batch_mixes_written_and_reduced():
    from paper_2601_01903_amd import BatchPlan
    ds = [20, 11, 13, 5, 14, 11, 18, 12, 15, 21, 16, 8]
    ls = [4, 4, 3, 2, 4, 1, 2, 4, 3, 4, 4, 1]
    say("[case] fold batch")
    vals = [values(d, 100 + i).astype(np.float32) for i, d in enumerate(ds)]
    x = torch.from_numpy(np.concatenate(vals)).to(DEV)
    bp = BatchPlan(ds, ls, dtype="f32")
    first = bp.apply(x)
    o = first.double().cpu().numpy()
    for i, (d, l) in enumerate(zip(ds, ls)):
        ref = oracle.fsi_c(vals[i].astype(np.float64), d, l, nthreads=16)
        assert normwise(o[bp.out_offset[i]:bp.out_offset[i + 1]], ref) < 1e-6, (d, l)
    for rep in range(4):
        s = float(1 << rep)
        y = x * s
        a, b = torch.full_like(first, float("nan")), torch.full_like(first, float("nan"))
        c = torch.full_like(first, float("nan"))
        bp.apply(y, out=a)
        bp.apply_noalloc(y, b)
        for st in range(bp.num_stages()):
            bp.apply_stage(y, c, st)
        torch.cuda.synchronize()
        for r in (a, b, c):
            assert torch.equal(r, first * s)
    bp.close()


def test_batch_of_one_item_instances_is_one_stage():
    from paper_2601_01903_amd import BatchPlan
    say("[case] fold batch, one stage")
    bp = BatchPlan([11, 9, 10], [3, 2, 4], dtype="f64")
    assert bp.num_stages() == 1
    bp.close()
