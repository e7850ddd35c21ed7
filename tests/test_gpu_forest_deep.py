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


@pytest.mark.parametrize("n_trees", [1, 6])
def test_cost_of_a_deep_tree(n_trees):
    """Trees of 2^14 leaves against trees of 2^6: the depths differ by 2.3."""
    d = 10
    x, bgs = np.ones(d), np.zeros((1, d))
    us = {}
    for depth in (6, 14):
        forest = full_trees(d, n_trees, depth, np.random.default_rng(depth))
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


def joined(a, b, at):
    """The trees of b after every at trees of a."""
    n = a[1].size
    roots = []
    take = iter(b[0])
    for k, r in enumerate(a[0]):
        roots.append(r)
        if k % at == at - 1:
            roots.extend(n + t for t in [next(take, None)] if t is not None)
    arrays = [np.concatenate([u, v]) for u, v in zip(a[1:], b[1:])]
    inner = b[1] >= 0
    for i in (2, 3):                        # children
        arrays[i][n:] = np.where(inner, b[i + 1] + n, 0)
    return (np.array(roots, np.int32), *[np.ascontiguousarray(x) for x in arrays])


# deep trees without a list among shallow ones that have one: one in 130 and in
# 40 of them (below and past the share at which every wave walks), in pairs, all
@pytest.mark.parametrize("d", [5, 9, 14, 16, 17, 18, 19, 21])
@pytest.mark.parametrize("shallow,deep,at", [(260, 2, 130), (200, 5, 40), (40, 40, 1), (1, 30, 1)])
def test_trees_without_a_list(d, shallow, deep, at):
    say(f"[case] overflow d={d} {deep} of {shallow + deep}")
    rng = np.random.default_rng(9400 + d)
    forest = joined(full_trees(d, shallow, 3, rng), full_trees(d, deep, 9, rng), at)
    x, bgs = np.ones(d), np.zeros((2, d))
    bgs[1] = rng.uniform(size=d)            # a background that decides some nodes
    got = gpu_values(d, forest, x, bgs, "f64")
    if d <= 9:
        assert np.array_equal(got, oracle.forest_values(d, *forest, x, bgs))
        return
    for S in np.concatenate([rng.integers(0, 1 << d, size=8), [0, (1 << d) - 1]]):
        assert got[S] == oracle.forest_value_at(int(S), d, *forest, x, bgs), int(S)


# ns per tree, background, level and coalition: plain walks take 0.0055 and
# 0.0007 at these sizes, the bounds are about twice that
@pytest.mark.parametrize("d,n_trees,depth,n_bg,bound", [(16, 50, 12, 2, 0.011), (20, 20, 12, 1, 0.0015)])
def test_cost_where_lists_overflow(d, n_trees, depth, n_bg, bound):
    forest = full_trees(d, n_trees, depth, np.random.default_rng(5))
    us = walk_us(d, forest, np.ones(d), np.zeros((n_bg, d)))
    say(f"[case] overflow cost d={d} depth={depth}: {us:.1f} us")
    assert us * 1e3 < bound * n_trees * n_bg * depth * 2 ** d


@pytest.mark.parametrize("d", [12, 17])
@pytest.mark.parametrize("n_trees,max_bg", [(60, 4096), (120, 600)])
def test_blocks_list_where_the_lists_find_no_room(n_trees, max_bg, d):
    """Forests made for so many backgrounds that they keep no lists, or lists of
    fewer than 64 leaves."""
    say(f"[case] forest without lists d={d} trees={n_trees}")
    rng = np.random.default_rng(43)
    forest = full_trees(d, n_trees, 6, rng)
    for x, bgs in ((rng.uniform(size=d), rng.uniform(size=(3, d))), (np.ones(d), np.zeros((2, d)))):
        got = gpu_values(d, forest, x, bgs, "f64", max_bg=max_bg)
        if d == 12:
            assert np.array_equal(got, oracle.forest_values(d, *forest, x, bgs))
            continue
        for S in np.concatenate([rng.integers(0, 1 << d, size=16), [0, (1 << d) - 1]]):
            assert got[S] == oracle.forest_value_at(int(S), d, *forest, x, bgs), int(S)


# both sides of the lines between the kernels: plain walks (up to 32 loads, 12 at
# d = 20, none past d = 23), and from d = 15 one or 64 coalitions a workgroup's lane
@pytest.mark.parametrize("d,n_trees,depth", [(1, 4, 2), (9, 32, 1), (9, 33, 1), (10, 4, 11), (10, 5, 11),
                                             (15, 16, 4), (15, 17, 4), (16, 64, 4), (16, 65, 4),
                                             (20, 12, 1), (20, 13, 1), (23, 1, 1), (24, 1, 1),
                                             (9, 3, 0), (9, 40, 0), (20, 13, 0)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_kernel_lines(d, n_trees, depth, dtype):
    say(f"[case] walk lines d={d} trees={n_trees} depth={depth} {dtype}")
    rng = np.random.default_rng(9500 + d)
    forest = full_trees(d, n_trees, depth, rng)
    x, bgs = rng.uniform(size=d), rng.uniform(size=(1, d))
    got = gpu_values(d, forest, x, bgs, dtype)
    cast = np.float64 if dtype == "f64" else np.float32
    if d <= 10:
        assert np.array_equal(got, oracle.forest_values(d, *forest, x, bgs).astype(cast))
        return
    for S in np.concatenate([rng.integers(0, 1 << d, size=16), [0, (1 << d) - 1]]):
        assert got[S] == cast(oracle.forest_value_at(int(S), d, *forest, x, bgs)), int(S)


def test_cost_of_few_trees():
    """Ten depth-3 trees: d = 16 is a quarter of d = 18."""
    us = {}
    for d in (16, 18):
        rng = np.random.default_rng(d)
        forest = full_trees(d, 10, 3, rng)
        us[d] = walk_us(d, forest, rng.uniform(size=d), rng.uniform(size=(1, d)))
        say(f"[case] few trees d={d}: {us[d]:.1f} us")
    assert us[16] < 1.6 * us[18]
