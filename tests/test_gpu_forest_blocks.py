"""GPU walk route of the value function (include/fsi_forest.h) at the sizes
where its blocks, leaf lists and chunks can go wrong: coalition counts around
the block sizes, trees whose reachable leaves outnumber a list, pair counts
around a chunk. Leaves are chosen by exact comparisons and summed in the
oracle's order, so every value is bitwise the oracle's."""
import numpy as np
import pytest

import oracle
from helpers import say
from test_gpu_forest import gpu_values, random_forest

pytestmark = pytest.mark.gpu


def full_trees(d, n_trees, depth, rng):
    """Heap-ordered full trees over random features, thresholds in (0, 1)."""
    inner, n = (1 << depth) - 1, (2 << depth) - 1
    feature = np.full((n_trees, n), -1, dtype=np.int32)
    feature[:, :inner] = rng.integers(0, d, size=(n_trees, inner))
    threshold = np.where(feature >= 0, rng.uniform(0.01, 0.99, size=feature.shape), 0.0)
    base = (np.arange(n_trees) * n)[:, None]
    idx = np.arange(n)[None, :]
    left = np.where(feature >= 0, base + 2 * idx + 1, 0).astype(np.int32)
    right = np.where(feature >= 0, base + 2 * idx + 2, 0).astype(np.int32)
    value = rng.standard_normal((n_trees, n))
    return (base[:, 0].astype(np.int32), feature.ravel(), threshold.ravel(), left.ravel(),
            right.ravel(), value.ravel())


# 5 .. 7: around one wave of coalitions; 15 .. 21: every kernel choice
@pytest.mark.parametrize("d", [2, 5, 6, 7, 10, 15, 16, 17, 18, 19, 21])
@pytest.mark.parametrize("undecided", [False, True])
def test_blocks_and_full_lists(d, undecided):
    """undecided: x = 1 and background 0, so that no node is decided by the
    points and a depth-7 tree overflows the leaf lists."""
    say(f"[case] forest blocks d={d} undecided={undecided}")
    rng = np.random.default_rng(9200 + d)
    forest = full_trees(d, 9, 7, rng)
    x = np.ones(d) if undecided else rng.uniform(size=d)
    bgs = np.zeros((1, d)) if undecided else rng.uniform(size=(3, d))
    got = gpu_values(d, forest, x, bgs, "f64", max_bg=3)
    if d <= 15:
        assert np.array_equal(got, oracle.forest_values(d, *forest, x, bgs))
        return
    picks = np.concatenate([rng.integers(0, 1 << d, size=48), [0, 1, 255, 256, (1 << d) - 1]])
    for S in picks:
        assert got[S] == oracle.forest_value_at(int(S), d, *forest, x, bgs), int(S)


# pairs = trees x backgrounds around the chunks of 256 and 512
@pytest.mark.parametrize("d,n_trees,n_bg", [(6, 1, 1), (7, 63, 1), (6, 51, 5), (9, 257, 1),
                                            (6, 171, 3), (6, 57, 9), (16, 17, 15), (16, 257, 1)])
def test_chunk_edges(d, n_trees, n_bg):
    say(f"[case] forest chunks d={d} trees={n_trees} n_bg={n_bg}")
    rng = np.random.default_rng(9300 + n_trees)
    x, bgs = rng.uniform(size=d), rng.uniform(size=(n_bg, d))
    forest = random_forest(d, n_trees, 5, rng, x, bgs)
    got = gpu_values(d, forest, x, bgs, "f64", max_bg=n_bg)
    if d <= 9:
        assert np.array_equal(got, oracle.forest_values(d, *forest, x, bgs))
        return
    for S in np.concatenate([rng.integers(0, 1 << d, size=24), [0, (1 << d) - 1]]):
        assert got[S] == oracle.forest_value_at(int(S), d, *forest, x, bgs), int(S)
