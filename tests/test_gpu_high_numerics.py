"""Numerics at the edges of the kernel of orders 5 and 6: values that are not
finite, and the two-float butterfly."""
import numpy as np
import pytest

import oracle
from helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype,prec", [("f64", "auto"), ("f32", "auto"), ("f32", "f32")])
@pytest.mark.parametrize("d,l", [(5, 5), (6, 5), (8, 6), (10, 5), (11, 6)])
def test_infinite_grand_coalition(d, l, dtype, prec):
    """v infinite at the full set only: a(full) is the one infinite coefficient,
    so a score it enters with weight W(s, d) is W times infinity, at sizes that
    the 11-bit tile pads as well."""
    from paper_2601_01903_amd import Plan
    say(f"[case] infinite value d={d} l={l} {dtype} {prec}")
    v = np.random.default_rng(d).standard_normal(1 << d)
    v[-1] = np.inf
    plan = Plan(d, l, dtype=dtype, precision=prec)
    assert plan.info()["tile_bits"] == 11
    x = torch.from_numpy(v).to(DEV, torch.float64 if dtype == "f64" else torch.float32)
    got = plan.apply(x).cpu().numpy()
    size = np.array([bin(int(m)).count("1") for m in oracle.output_masks(d, l)])
    for s in range(l + 1):
        w = oracle.index_weight_exact("fsi", s, d, l)
        if w != 0:
            assert (got[size == s] == np.inf * (1 if w > 0 else -1)).all(), s
    plan.close()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("d,l", [(9, 5), (12, 5), (13, 6)])
def test_infinite_coefficient_below(d, l, dtype):
    """Moebius input with a(empty set) infinite: the empty set is a superset of
    itself only, so every other score stays finite."""
    from paper_2601_01903_amd import Plan
    say(f"[case] infinite coefficient d={d} l={l} {dtype}")
    a = np.random.default_rng(d).standard_normal(1 << d)
    a[0] = np.inf
    plan = Plan(d, l, dtype=dtype, input="mobius")
    x = torch.from_numpy(a).to(DEV, torch.float64 if dtype == "f64" else torch.float32)
    got = plan.apply(x).cpu().numpy()
    assert np.isinf(got[0]) and np.isfinite(got[1:]).all()
    plan.close()


def two_float_moebius(v, order):
    """Butterfly over the bits in this order in renormalised pairs of FP32."""
    f = np.float32
    hi, lo = v.astype(f), np.zeros(v.size, f)
    for i in order:
        h, w = hi.reshape(-1, 2, 1 << i), lo.reshape(-1, 2, 1 << i)
        a, b = h[:, 1].copy(), -h[:, 0]
        s = a + b
        t = s - a
        e = ((a - (s - t)) + (b - t)) + (w[:, 1] - w[:, 0])
        h[:, 1] = s + e
        w[:, 1] = e - (h[:, 1] - s)
    return hi + lo


@pytest.mark.parametrize("seed", [0, 1])
def test_two_float_form_is_renormalised(seed):
    """Large values that cancel in every coefficient, beside values near their
    last bit: the low words carry the result. The scores of 2 to 5 players of
    the Shapley-Taylor index of order 6 are the coefficients themselves, rounded
    once, in the kernel's order of the bits."""
    from paper_2601_01903_amd import Plan
    d, l = 11, 6
    say(f"[case] two-float form seed={seed}")
    S = np.arange(1 << d)
    big = ((S[:, None] >> np.arange(d)) & 1) @ (1 - 2 * (np.arange(d) % 2)) * 2500001.0
    small = np.random.default_rng(seed).standard_normal(1 << d) * 2.0 ** -5
    v = np.where(big != 0, big, small).astype(np.float32)
    plan = Plan(d, l, dtype="f32", precision="f32_compensated", index="stii")
    assert plan.info()["tile_bits"] == 11
    got = plan.apply(torch.from_numpy(v).to(DEV)).cpu().numpy()
    masks = oracle.output_masks(d, l).astype(np.int64)
    size = np.array([bin(int(m)).count("1") for m in masks])
    keep = (size >= 2) & (size < l)
    want = two_float_moebius(v, [8, 9, 10, 4, 5, 6, 7, 0, 1, 2, 3])
    assert (got[keep] == want[masks[keep]]).all()
    plan.close()
