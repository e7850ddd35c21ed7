"""GPU Moebius route of the value function (include/fsi_forest.h): the shared
lists of the scatter at the edges of their chunks of 256 paths and groups of
backgrounds, and every number of bits a pass of the subset sums can take. Leaf
outputs are multiples of 2^-10, so the sums are exact and the route's values are
bitwise the walk's (as long as the division by the backgrounds is exact too)."""
import numpy as np
import pytest

from helpers import normwise, say
from test_gpu_forest_blocks import full_trees

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def both_routes(d, n_trees, depth, n_bg, dtype, undecided=False, time=False):
    from paper_2601_01903_amd import Forest
    rng = np.random.default_rng([d, n_trees, n_bg])
    forest = list(full_trees(d, n_trees, depth, rng))
    forest[5] = np.round(forest[5] * 1024) / 1024
    x = np.ones(d) if undecided else rng.uniform(size=d)
    bgs = np.zeros((n_bg, d)) if undecided else rng.uniform(size=(n_bg, d))
    F = Forest(d, *forest, max_bg=n_bg)
    xd, bd = torch.as_tensor(x).to(DEV), torch.as_tensor(bgs).to(DEV)
    walk = F.values(xd, bd, dtype=dtype).cpu().numpy()
    moeb = F.values(xd, bd, dtype=dtype, method="mobius").cpu().numpy()
    us = np.inf
    if time:
        work, out = (torch.empty(1 << d, dtype=torch.float64, device=DEV) for _ in range(2))
        for _ in range(10):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda.synchronize()
            e[0].record()
            for _ in range(10):
                F.values(xd, bd, out=out, method="mobius", work=work)
            e[1].record()
            torch.cuda.synchronize()
            us = min(us, e[0].elapsed_time(e[1]) * 100)
    F.close()
    return walk, moeb, us


# one pass up to d = 12, one high pass of 1 to 8 bits to d = 20, two past that
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("d", [1, 2, 5, 11, 12, 13, 14, 15, 16, 17, 18, 19, 20, 21, 23])
def test_passes_bitwise(d, dtype):
    say(f"[case] subset sums d={d} {dtype}")
    walk, moeb, _ = both_routes(d, 12, 5, 8, dtype)
    assert np.array_equal(walk, moeb)


# 9 trees are 288 paths (two chunks), 60 are 8 chunks: groups of 1, 2, 4 and 8
@pytest.mark.parametrize("undecided", [False, True])
@pytest.mark.parametrize("n_trees,n_bg", [(1, 1), (8, 9), (9, 1), (9, 7), (9, 16), (60, 5), (60, 8),
                                          (60, 9), (60, 20), (60, 40), (60, 64)])
def test_chunks_and_groups(n_trees, n_bg, undecided):
    say(f"[case] scatter trees={n_trees} n_bg={n_bg} undecided={undecided}")
    walk, moeb, _ = both_routes(10, n_trees, 5, n_bg, "f64", undecided)
    if n_bg & (n_bg - 1) == 0:
        assert np.array_equal(walk, moeb)
    else:
        assert normwise(moeb, walk) < 1e-12


def test_cost_of_few_paths():
    """Ten depth-5 trees with every path reachable: eight backgrounds against one."""
    us = {n_bg: both_routes(16, 10, 5, n_bg, "f64", undecided=True, time=True)[2] for n_bg in (1, 8)}
    say(f"[case] few paths: {us[1]:.1f}, {us[8]:.1f} us")
    assert us[8] < 1.6 * us[1]
