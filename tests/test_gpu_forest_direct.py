"""The direct forest walk where its tiling can go wrong: every depth, tree
counts around a group of trees, row counts around a tile and a round of tiles,
both tile heights.  Scores are compared with the binary64 sum of the leaves
that the leaf kernel walks to, and with the scores of the same rows in other
calls, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


def make(seed, R, F, trees, depth, flags, ld):
    g = np.random.default_rng(seed)
    X = g.integers(-20, 21, (R, ld)).astype(np.float32)
    X[g.random((R, ld)) < 0.01] = np.nan
    X[g.random((R, ld)) < 0.01] = -np.inf
    n_int = (1 << depth) - 1
    thr = g.integers(-20, 21, (trees, n_int)).astype(np.float32)
    thr[g.random(thr.shape) < 0.01] = np.nan                  # the direct walk takes them: never less
    thr[g.random(thr.shape) < 0.01] = -np.inf
    f = dict(n_trees=trees, depth=depth, n_features=F, flags=flags, base_score=0.25,
             # a feature past the last column reads the last column
             node_feature=g.integers(0, min(F + 2, 256), (trees, n_int)).astype(np.uint8), node_threshold=thr,
             leaf_value=g.normal(0, 1, (trees, 1 << depth)).astype(np.float32))
    d = {k: (hwsel.to_device(v) if isinstance(v, np.ndarray) else v) for k, v in f.items()}
    return f, d, torch.from_numpy(X).cuda()


def check(f, d, X):
    R, T = X.shape[0], f["n_trees"]
    got = hwsel.hwsel_forest_score(d, X)
    at = torch.arange(R, device="cuda")
    if R > 5000:                                              # both ends and a spread between
        at = torch.cat([at[:700], at[700:-700:61], at[-700:]])
    leaves = hwsel.hwsel_forest_leaves(d, X, at).cpu().numpy().view(np.uint16)
    v = f["leaf_value"].astype(np.float64)[np.arange(T)[None, :], leaves.astype(np.int64)]
    # any order of n fp32 additions is within n 2^-24 of the terms' magnitudes
    bound = (T + 1) * 2.0 ** -24 * (f["base_score"] + np.abs(v).sum(1))
    assert np.all(np.abs(got[at].cpu().numpy() - (f["base_score"] + v.sum(1))) <= bound)
    few = min(R, 301)
    assert torch.equal(hwsel.hwsel_forest_score(d, X[R - few:].contiguous()), got[R - few:])


@pytest.mark.parametrize("depth", range(1, 13))
def test_every_depth(depth):
    group = 8 if depth >= 11 else 16 if depth == 10 else 32
    for i, (R, F, T) in enumerate([(1, 1, 1), (15, 128, group - 1), (2049, 33, group), (2200, 129, group + 1),
                                   (2303, 256, 2 * group + 3), (2500, 128, 3 * group)]):
        say(f"depth {depth}: {R} rows, {F} features, {T} trees")
        check(*make(100 * depth + i, R, F, T, depth, i % 2, F + (3 if i % 3 else 0)))


@pytest.mark.parametrize("R", [2047, 2048, 32767, 32769, 34816, 34817, 65537])
def test_rounds(R):
    """Rows at the edges of a round of 256 tiles, with and without rows left
    to single waves; more trees than one pass of those."""
    for F, T, depth in ((40, 300, 6), (200, 20, 11)):
        say(f"{R} rows, {F} features, {T} trees of depth {depth}")
        check(*make(R, R, F, T, depth, 1, F))


@pytest.mark.parametrize("offset", [1, 2, 3])
@pytest.mark.parametrize("depth", [1, 2, 7, 9, 11])
def test_feature_bytes_anywhere(offset, depth):
    """Feature bytes that begin inside a word: they are copied as whole words."""
    say(f"depth {depth}, features {offset} bytes into a word")
    f, d, X = make(depth, 5000, 70, 37, depth, 1, 70)
    want = hwsel.hwsel_forest_score(d, X)
    flat = d["node_feature"].reshape(-1)
    moved = torch.zeros(flat.numel() + 4, dtype=torch.uint8, device="cuda")
    moved[offset:offset + flat.numel()] = flat
    d["node_feature"] = moved[offset:offset + flat.numel()].view(d["node_feature"].shape)
    assert d["node_feature"].data_ptr() % 4 == offset
    check(f, d, X)
    assert torch.equal(hwsel.hwsel_forest_score(d, X), want)


@pytest.mark.parametrize("T,depth", [(1, 1), (1, 12), (2, 6), (3, 4), (4, 6), (5, 5), (6, 4), (7, 3), (8, 3), (9, 4), (8, 8),
                                     (16, 4), (13, 5)])
def test_few_trees(T, depth):
    """Around the numbers of node visits that a row per thread takes: the same
    rows go another way in a call of another length, with the same bits."""
    for R, F in ((4096, 1), (4097, 31), (32768, 32), (32769, 32), (33000, 33), (5000, 128), (5000, 129), (40000, 5)):
        say(f"{T} trees of depth {depth}, {R} rows, {F} features")
        check(*make(R + T, R, F, T, depth, T % 2, F + T % 4))


def test_more_rows_than_one_launch_holds():
    """Past 2^29 rows the tiles' threads, eight a row, no longer fit one launch."""
    R, T, depth = (1 << 29) + 777, 22, 3
    g = np.random.default_rng(9)
    f = dict(n_trees=T, depth=depth, n_features=1, flags=0, base_score=0.5,
             node_feature=np.zeros((T, 7), np.uint8), node_threshold=g.normal(0, 1, (T, 7)).astype(np.float32),
             leaf_value=g.normal(0, 1, (T, 8)).astype(np.float32))
    d = {k: (hwsel.to_device(v) if isinstance(v, np.ndarray) else v) for k, v in f.items()}
    X = torch.randn(R, 1, device="cuda")
    say(f"{R} rows")
    got = hwsel.hwsel_forest_score(d, X)
    for lo in (0, (1 << 28) - 500, (1 << 29) - 500, R - 1000):
        assert torch.equal(hwsel.hwsel_forest_score(d, X[lo:lo + 1000]), got[lo:lo + 1000])
    del X, got
    torch.cuda.empty_cache()
