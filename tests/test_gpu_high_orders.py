"""Register-phase kernel of orders 5 and 6: every size from d = l up through
the first multi-tile ones, the storage and precision forms, Moebius input and
the other indices, single and in batches beside the other kernels, against the
C oracle."""
import numpy as np
import pytest

import games
import oracle
from helpers import normwise, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def values(d, seed):
    return games.tree_values(games.tree_game(d, 30, 5, games.rng_for(961, seed)))


@pytest.mark.parametrize("dtype,prec,tol", [("f64", "auto", 1e-12), ("f32", "auto", 1e-6),
                                            ("f32", "f32_compensated", 1e-6), ("f32", "f32", 2e-6)])
@pytest.mark.parametrize("l", [5, 6])
@pytest.mark.parametrize("d", [6, 9, 11, 12, 13, 15, 16])
def test_single(d, l, dtype, prec, tol):
    from paper_2601_01903_amd import Plan
    say(f"[case] high order d={d} l={l} {dtype} {prec}")
    v = values(d, d).astype(np.float64 if dtype == "f64" else np.float32)
    ref = oracle.fsi_c(v.astype(np.float64), d, l, nthreads=16)
    plan = Plan(d, l, dtype=dtype, precision=prec)
    assert plan.info()["tile_bits"] == 11
    x = torch.from_numpy(v).to(DEV)
    a = plan.apply(x)
    b = plan.apply(x * 2)
    assert torch.equal(b, a * 2)
    assert normwise(a.double().cpu().numpy(), ref) < tol
    gen = Plan(d, l, dtype=dtype, precision=prec, kernel="generic")
    assert normwise(gen.apply(x).double().cpu().numpy(), ref) < tol
    plan.close()
    gen.close()


@pytest.mark.parametrize("index", ["stii", "sii", "ksii", "bii"])
def test_indices_and_moebius_input(index):
    from paper_2601_01903_amd import Plan
    for d, l in [(9, 5), (13, 6)]:
        say(f"[case] high order {index} d={d} l={l}")
        v = values(d, 50 + d)
        ref = oracle.interaction(v, d, l, index)
        x = torch.from_numpy(v).to(DEV)
        got = Plan(d, l, dtype="f64", index=index).apply(x)
        assert normwise(got.cpu().numpy(), ref) < 1e-12
        a = Plan(d, 1, dtype="f64").mobius(x.clone())
        got = Plan(d, l, dtype="f64", index=index, input="mobius").apply(a)
        assert normwise(got.cpu().numpy(), ref) < 1e-12


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-6)])
def test_batch_beside_the_other_kernels(dtype, tol):
    from paper_2601_01903_amd import BatchPlan
    ds = [13, 12, 9, 16, 11, 14, 17, 10, 15, 8]
    ls = [5, 4, 7, 6, 5, 2, 5, 6, 6, 3]
    say(f"[case] high order batch {dtype}")
    np_t = np.float64 if dtype == "f64" else np.float32
    vals = [values(d, 100 + i).astype(np_t) for i, d in enumerate(ds)]
    x = torch.from_numpy(np.concatenate(vals)).to(DEV)
    bp = BatchPlan(ds, ls, dtype=dtype)
    first = bp.apply(x)
    o = first.double().cpu().numpy()
    for i, (d, l) in enumerate(zip(ds, ls)):
        ref = oracle.fsi_c(vals[i].astype(np.float64), d, l, nthreads=16)
        assert normwise(o[bp.out_offset[i]:bp.out_offset[i + 1]], ref) < tol, (d, l)
    for s in (2.0, 1.0):
        y = x * s
        a, b, c = (torch.full_like(first, float("nan")) for _ in range(3))
        bp.apply(y, out=a)
        bp.apply_noalloc(y, b)
        for st in range(bp.num_stages()):
            bp.apply_stage(y, c, st)
        torch.cuda.synchronize()
        for r in (a, b, c):
            assert torch.equal(r, first * s)
    bp.close()


@pytest.mark.parametrize("n,d,l", [(2700, 9, 5), (1300, 7, 6), (70, 16, 6)])
def test_scratch_bound(n, d, l):
    """Batches whose results of the register phases exceed the 64 MiB of the
    call without allocation: the generic kernel where its results fit, so that
    the call takes the plan; else the register phases, and the call refuses."""
    from paper_2601_01903_amd import BatchPlan, FsiError
    say(f"[case] high order scratch {n} x d={d} l={l}")
    v = np.concatenate([values(d, 300 + i) for i in range(4)]).astype(np.float32)
    x = torch.from_numpy(v).to(DEV).repeat(n // 4 + 1)[: n << d].contiguous()
    bp = BatchPlan([d] * n, [l] * n, dtype="f32")
    out = bp.apply(x)
    m = bp.out_offset[1]
    for i in range(4):
        ref = oracle.fsi_c(v[i << d:(i + 1) << d].astype(np.float64), d, l, nthreads=16)
        assert normwise(out[i * m:(i + 1) * m].double().cpu().numpy(), ref) < 1e-6
        assert torch.equal(out[i * m:(i + 1) * m], out[(i + n // 4 * 4 - 4) * m:][:m])
    got = torch.full_like(out, float("nan"))
    if d <= 11:
        bp.apply_noalloc(x, got)
        assert torch.equal(got, out)
    else:
        with pytest.raises(FsiError, match="scratch"):
            bp.apply_noalloc(x, got)
    bp.close()


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-12), ("f32", 1e-6)])
@pytest.mark.parametrize("n", [256, 260])
def test_many_small_instances(n, dtype, tol):
    """On both sides of the line (one instance per CU) between the kernels."""
    from paper_2601_01903_amd import BatchPlan
    say(f"[case] high order small {n} {dtype}")
    np_t = np.float64 if dtype == "f64" else np.float32
    ds = [6, 7, 8, 9, 10] * (n // 5) + [6] * (n % 5)
    ls = [5 + i % 2 for i in range(n)]
    game = {d: values(d, 400 + d).astype(np_t) for d in set(ds)}
    x = torch.from_numpy(np.concatenate([game[d] for d in ds])).to(DEV)
    refs = {(d, l): oracle.fsi_c(game[d].astype(np.float64), d, l, nthreads=16)
            for d, l in set(zip(ds, ls))}
    bp = BatchPlan(ds, ls, dtype=dtype)
    o = bp.apply(x).double().cpu().numpy()
    for i, (d, l) in enumerate(zip(ds, ls)):
        assert normwise(o[bp.out_offset[i]:bp.out_offset[i + 1]], refs[d, l]) < tol, (i, d, l)
    bp.close()
