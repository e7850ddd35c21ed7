"""The Moebius butterfly (fsi_mobius) at the sizes where its passes change: one
low pass of up to 12 bits, then one strided pass per 8 bits above them, of 1 to
8 bits each. Integer values whose transform stays below the significand are
transformed exactly, so the result is the integer butterfly's, bit for bit."""
import numpy as np
import pytest

from helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def int_mobius(v, d):
    a = v.copy()
    for i in range(d):
        x = a.reshape(-1, 2, 1 << i)
        x[:, 1] -= x[:, 0]
    return a


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("d", [1, 3, 4, 5, 8, 11, 12, 13, 14, 16, 17, 18, 19, 20, 21, 23])
def test_every_pass_size(d, dtype):
    say(f"[case] moebius passes d={d} {dtype}")
    from paper_2601_01903_amd import Plan
    rng = np.random.default_rng(940 + d)
    # |a| <= 2^d max|v|: below 2^53, and below 2^24 with values that vanish
    # but on 2^3 sets
    if dtype == "f64":
        v = rng.integers(-1000, 1000, size=1 << d).astype(np.int64)
    else:
        v = np.zeros(1 << d, dtype=np.int64)
        v[rng.integers(0, 1 << d, size=8)] = rng.integers(-1000, 1000, size=8)
    tdt = torch.float64 if dtype == "f64" else torch.float32
    a = torch.from_numpy(v).to(DEV).to(tdt)
    plan = Plan(d, 1, dtype=dtype)
    plan.mobius(a)
    got = a.double().cpu().numpy()
    plan.close()
    assert np.array_equal(got, int_mobius(v, d).astype(np.float64))


@pytest.mark.parametrize("precision", ["f32", "f32_compensated", "auto"])
def test_two_pass_batch_of_uneven_sizes(precision):
    """One batch whose instances take no, one and two high passes and start
    at every alignment; against each instance planned alone with the fused
    algorithm (both within the FP32 form's 1e-6 of the FP64 result)."""
    say(f"[case] two-pass uneven sizes {precision}")
    from paper_2601_01903_amd import BatchPlan, Plan
    ds, ls = [1, 2, 13, 3, 12, 21, 5, 16, 20], [1, 1, 2, 2, 3, 1, 2, 2, 2]
    bp = BatchPlan(ds, ls, dtype="f32", precision=precision, algo="two_pass")
    g = torch.Generator().manual_seed(941)
    v = torch.rand(bp.value_offset[-1], generator=g, dtype=torch.float32)
    # smooth games: a small random part on an additive one
    parts = []
    for d, o in zip(ds, bp.value_offset):
        idx = torch.arange(1 << d)
        pop = sum(((idx >> i) & 1) for i in range(d)).float()
        parts.append(pop + 1e-3 * v[o:o + (1 << d)])
    v = torch.cat(parts).to(DEV)
    out = bp.apply(v)
    for i, (d, l) in enumerate(zip(ds, ls)):
        ref = Plan(d, l, dtype="f64").apply(
            v[bp.value_offset[i]:bp.value_offset[i + 1]].double().contiguous())
        got = out[bp.out_offset[i]:bp.out_offset[i + 1]].double()
        # the transform of 1e-3 uniform noise reaches 1e-3 * 2^(d / 2), and
        # FP32 forms round it at 2^-24 through at most 2 d additions
        tol = 2 * d * 2.0 ** -24 * (d + 1e-3 * 2.0 ** (d / 2 + 3))
        assert float((got - ref).abs().max()) <= tol, (d, l)
    bp.close()
