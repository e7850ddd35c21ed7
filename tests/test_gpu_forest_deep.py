"""GPU walk route of the value function on deep trees (include/fsi_forest.h):
bitwise the oracle's values, at a cost that follows the depth and not the
number of root-to-leaf paths."""
import numpy as np
import pytest

import oracle
from helpers import say
from test_gpu_forest import gpu_values
from test_gpu_forest_blocks import full_trees

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def walk_us(d, forest, x, bgs):
    from paper_2601_01903_amd import Forest
    F = Forest(d, *forest, max_bg=len(bgs))
    xd, bd = (torch.as_tensor(a).to("cuda:0") for a in (x, np.ascontiguousarray(bgs)))
    out = torch.empty(1 << d, dtype=torch.float64, device="cuda:0")
    best = np.inf
    for _ in range(10):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        torch.cuda.synchronize()
        e[0].record()
        for _ in range(10):
            F.values(xd, bd, dtype="f64", out=out)
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 100)
    F.close()
    return best


def test_cost_of_a_deep_tree():
    """One tree of 2^14 leaves against one of 2^6: the depths differ by 2.3."""
    d = 10
    x, bgs = np.ones(d), np.zeros((1, d))
    us = {}
    for depth in (6, 14):
        forest = full_trees(d, 1, depth, np.random.default_rng(depth))
        assert np.array_equal(gpu_values(d, forest, x, bgs), oracle.forest_values(d, *forest, x, bgs))
        us[depth] = walk_us(d, forest, x, bgs)
        say(f"[case] deep tree d={d} depth={depth}: {us[depth]:.1f} us")
    assert us[14] < 12 * us[6]


@pytest.mark.parametrize("undecided", [False, True])
def test_shared_nodes(undecided):
    """Layers of three nodes that share their children: 2^20 paths of 60 nodes."""
    d, levels, width = 12, 20, 3
    say(f"[case] shared nodes undecided={undecided}")
    rng = np.random.default_rng(41)
    n = (levels + 1) * width
    feature = rng.integers(0, d, n).astype(np.int32)
    feature[-width:] = -1
    below = lambda: np.minimum((np.arange(n) // width + 1) * width + rng.integers(0, width, n),
                               n - 1).astype(np.int32)
    forest = (np.arange(3, dtype=np.int32), feature, rng.uniform(0.01, 0.99, n), below(), below(),
              rng.standard_normal(n))
    x = np.ones(d) if undecided else rng.uniform(size=d)
    bgs = np.zeros((1, d)) if undecided else rng.uniform(size=(2, d))
    assert np.array_equal(gpu_values(d, forest, x, bgs), oracle.forest_values(d, *forest, x, bgs))
