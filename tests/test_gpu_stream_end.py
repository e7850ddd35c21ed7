"""Plans that outlive the stream they ran on: the stream goes right after the
apply, then the plan, and the scores are those of the default stream."""
import ctypes

import numpy as np
import pytest

from helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Stream:
    def __init__(self, lib):
        self.lib, h = lib, ctypes.c_void_p()
        assert lib.hipStreamCreateWithFlags(ctypes.byref(h), 1) == 0      # non-blocking
        self.cuda_stream = h.value

    def destroy(self):
        assert self.lib.hipStreamDestroy(ctypes.c_void_p(self.cuda_stream)) == 0


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("ds,ls", [([9], [2]), ([16, 12, 14], [4, 3, 6])])
def test_stream_destroyed_before_the_plan(ds, ls, graph):
    from paper_2601_01903_amd import BatchPlan, fsi
    say(f"[case] stream end {ds} graph={graph}")
    rng = np.random.default_rng(len(ds))
    v = torch.from_numpy(rng.standard_normal(sum(1 << d for d in ds))).to("cuda:0")
    plan = BatchPlan(ds, ls, dtype="f64")
    want = plan.apply(v).clone()
    torch.cuda.synchronize()
    for _ in range(3):
        p, s = BatchPlan(ds, ls, dtype="f64"), Stream(fsi.load())
        out = torch.full_like(want, float("nan"))
        torch.cuda.synchronize()
        p.apply(v, out=out, stream=s, graph=graph)
        s.destroy()
        p.close()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    plan.close()
