"""The register-phase kernel's forms: per order, few or all gather positions,
held registers with shared or separate LDS regions (batches of more work items
than CUs), against the C oracle on sampled instances, at the sizes on both
sides of each form's line."""
import numpy as np
import pytest

import games
import oracle
from helpers import normwise, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# l = 3: up to 4 positions (d <= 21) run the shared-region form; l = 4: up to
# 7 positions (d <= 17) the one with fewer accumulators
@pytest.mark.parametrize("dtype,prec,tol", [("f64", "auto", 1e-12), ("f32", "auto", 1e-6),
                                            ("f32", "f32_compensated", 1e-6), ("f32", "f32", 2e-6)])
@pytest.mark.parametrize("d,l,n", [(12, 1, 300), (13, 2, 300), (9, 3, 260), (12, 3, 300),
                                   (16, 3, 270), (11, 4, 300), (17, 4, 34), (18, 4, 20),
                                   (21, 3, 2), (22, 3, 2)])
def test_forms(d, l, n, dtype, prec, tol):
    from paper_2601_01903_amd import BatchPlan
    say(f"[case] forms d={d} l={l} n={n} {dtype} {prec}")
    np_t = np.float64 if dtype == "f64" else np.float32
    pool = [games.tree_values(games.tree_game(d, 30, 5, games.rng_for(971 + d, i))).astype(np_t)
            for i in range(2)]
    refs = [oracle.fsi_c(v.astype(np.float64), d, l, nthreads=16) for v in pool]
    x = torch.cat([torch.from_numpy(pool[i % 2]) for i in range(n)]).to(DEV)
    bp = BatchPlan([d] * n, [l] * n, dtype=dtype, precision=prec)
    out = bp.apply(x)
    again = bp.apply(x * 2)
    assert torch.equal(again, out * 2)
    o = out.double().cpu().numpy().reshape(n, -1)
    for i in range(n):   # every instance: equal games, equal bits
        assert np.array_equal(o[i], o[i % 2])
    for i in range(min(n, 2)):
        assert normwise(o[i], refs[i]) < tol
    bp.close()


@pytest.mark.parametrize("index", ["sii", "ksii"])
def test_forms_moebius_input(index):
    """Moebius input on the shared-region form."""
    from paper_2601_01903_amd import BatchPlan, Plan
    d, l, n = 12, 3, 280
    say(f"[case] forms moebius input {index}")
    v = games.tree_values(games.tree_game(d, 30, 5, games.rng_for(972, 0)))
    ref = oracle.interaction(v, d, l, index)
    a = Plan(d, l, dtype="f64").mobius(torch.from_numpy(v).to(DEV))
    for dtype, tol in (("f64", 1e-12), ("f32", 1e-6)):
        bp = BatchPlan([d] * n, [l] * n, dtype=dtype, index=index, input="mobius")
        x = a.to(torch.float64 if dtype == "f64" else torch.float32).repeat(n)
        o = bp.apply(x).double().cpu().numpy().reshape(n, -1)
        assert all(np.array_equal(o[i], o[0]) for i in range(n))
        assert normwise(o[0], ref) < tol
        bp.close()
