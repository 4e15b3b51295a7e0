"""The packed traversal where its tiling can go wrong: every depth, tree counts
around a chunk, row counts around a slice, a tile and the deferred-leaf tiles,
bin rows of every width.  Leaves are compared index by index with the direct
walk, scores with the binary64 sum of the very leaves."""
import numpy as np
import pytest
import torch

from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


def make(seed, R, F, trees, depth, flags=1):
    g = np.random.default_rng(seed)
    X = g.integers(-20, 21, (R, F)).astype(np.float32)
    X[g.random((R, F)) < 0.01] = np.nan
    X[g.random((R, F)) < 0.01] = np.inf
    n_int = (1 << depth) - 1
    f = dict(n_trees=trees, depth=depth, n_features=F, flags=flags, base_score=0.25,
             node_feature=g.integers(0, F, (trees, n_int)).astype(np.uint8),
             node_threshold=g.integers(-20, 21, (trees, n_int)).astype(np.float32),
             leaf_value=g.normal(0, 1, (trees, 1 << depth)).astype(np.float32))
    d = {k: (hwsel.to_device(v) if isinstance(v, np.ndarray) else v) for k, v in f.items()}
    return f, d, torch.from_numpy(X).cuda()


def check(f, d, X):
    R, T = X.shape[0], f["n_trees"]
    packed = hwsel.hwsel_forest_pack(d)
    rows = torch.arange(R, device="cuda")
    want = hwsel.hwsel_forest_leaves(d, X, rows).cpu().numpy().view(np.uint16)
    got = hwsel.hwsel_forest_score(d, X, packed=packed)
    checked, _, leaves = hwsel.hwsel_forest_score_checked(d, X, packed, leaf_rows=(0, R))
    assert np.array_equal(leaves.cpu().numpy().view(np.uint16), want)
    assert torch.equal(got, checked)
    v = f["leaf_value"].astype(np.float64)[np.arange(T)[None, :], want.astype(np.int64)]
    exact = f["base_score"] + v.sum(1)
    # any order of n fp32 additions is within n 2^-24 of the terms' magnitudes
    bound = (T + 1) * 2.0 ** -24 * (f["base_score"] + np.abs(v).sum(1))
    assert np.all(np.abs(got.cpu().numpy() - exact) <= bound)


@pytest.mark.parametrize("depth", range(1, 11))
def test_every_depth(depth):
    tc = 64 if depth <= 8 else 32
    for i, (R, F, T) in enumerate([(1, 1, 1), (17, 16, tc - 1), (255, 31, tc), (256, 64, tc + 1), (257, 96, 2 * tc),
                                   (300, 128, tc // 2 + 1)]):
        say(f"depth {depth}: {R} rows, {F} features, {T} trees")
        check(*make(100 * depth + i, R, F, T, depth, flags=i % 2))


@pytest.mark.parametrize("depth,R", [(10, 2047), (10, 2048), (10, 2049), (10, 4352 + 15), (9, 4097), (8, 4097),
                                     (8, 70_001), (10, 40_001), (10, 70_001), (10, 150_001)])
def test_tiles_and_groups(depth, R):
    """Rows at the edges of the deferred-leaf tiles, row groups across the XCDs
    (more than 2 MB of bins) with a ragged end, and items of one, up to four and
    more tiles (the checked walk always defers eight)."""
    say(f"depth {depth}: {R} rows")
    check(*make(R, R, 40 if R < 10_000 else 128, 70, depth))
