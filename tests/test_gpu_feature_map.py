"""The feature map where its arithmetic or its sharing of problem terms changes:
rows whose integers pass 2^50 (64-bit arithmetic instead of exact doubles),
hardware fields beyond the double path, segments of one row and runs of empty
ones, matrices past the last-level cache, and the fused binning of all of them
against features -> forest."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


def make(seed, lens, big=0):
    """Problems with the given segment lengths; every `big`-th one has M, N and
    K near 2^20 (their product, not its double, is below 2^62)."""
    g = np.random.default_rng(seed)
    P, R = len(lens), int(np.sum(lens))
    probs = np.zeros(P, synth.PROBLEM_DTYPE)
    for f in ("M", "N", "K"):
        probs[f] = np.exp(g.uniform(0, np.log(100_000), P)).astype(np.int32)
        if big:
            probs[f][::big] = g.integers((1 << 20) - 70, 1 << 20, len(probs[f][::big]))
    probs["layout"], probs["dtype"] = g.integers(0, 5, P), g.integers(0, 4, P)
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    pick = lambda *v: g.choice(v, R)  # noqa: E731
    c = dict(tile_m=pick(0, 1, 48, 64, 128, 192, 256, 333), tile_n=pick(1, 16, 80, 96, 256, 257), tile_k=pick(1, 32, 64, 96, 512),
             inst_n=pick(0, 8, 16, 48, 64, 256), stages=pick(0, 1, 2, 5, 12, 255), cluster_m=pick(0, 1, 2, 3, 16),
             cluster_n=pick(0, 1, 2, 5, 16), swizzle=pick(0, 1, 4), inst_m_div16=pick(0, 1, 4, 255), inst_k=pick(0, 7, 16, 32),
             kernel_sched=pick(0, 1, 2, 3), epi_sched=pick(0, 1, 2, 9), tile_sched=pick(0, 1, 2))
    return probs, seg, {n: c[n].astype(t) for n, t in synth.CAND_FIELDS}


def device(probs, seg, c):
    return (hwsel.to_device(probs), hwsel.to_device(seg), {n: hwsel.to_device(v) for n, v in c.items()})


HW = synth.hardware()
LENS = {"one row each": np.ones(700, int), "empty runs": np.array([3] + [0] * 300 + [70, 0, 1] + [0] * 40 + [500, 2]),
        "short": np.array([5, 17, 31, 64, 1] * 20), "one problem": np.array([1027]), "single row": np.array([1])}


@pytest.mark.parametrize("F", [64, 96, 128])
@pytest.mark.parametrize("case", list(LENS))
@pytest.mark.parametrize("big,hw", [(0, HW), (3, HW), (0, dict(HW, llc_bytes=(1 << 40) + 1))],
                         ids=["plain", "wide rows", "wide hardware"])
def test_columns_are_the_oracles(F, case, big, hw):
    say(f"{case}: F={F} big={big} llc={hw['llc_bytes']}")
    probs, seg, c = make(F + big, LENS[case], big)
    want = oracle.features(hw, probs, seg, c, F)
    dp, ds, dc = device(probs, seg, c)
    X = torch.full((int(seg[-1]), F + 4), -7.0, device="cuda")
    hwsel.hwsel_features(hw, dp, ds, dc, F, X=X)
    got = X.cpu().numpy()
    assert np.array_equal(got[:, :F].view(np.uint32), want.view(np.uint32)), np.argwhere(got[:, :F] != want)[:5]
    assert np.all(got[:, F:] == -7.0)
    # fused: a forest on the first nf columns, with an infinite threshold
    g = np.random.default_rng(5)
    for nf in (F, F - 13):
        T, D = 9, 4
        feat = g.integers(0, nf, (T, 15))
        thr = want[g.integers(0, len(want), (T, 15)), feat].astype(np.float32)
        thr[0, 3] = np.inf
        f = dict(n_trees=T, depth=D, n_features=nf, flags=1, base_score=0.0,
                 node_feature=hwsel.to_device(feat.astype(np.uint8)), node_threshold=hwsel.to_device(thr),
                 leaf_value=hwsel.to_device(g.normal(0, 1, (T, 16)).astype(np.float32)))
        packed = hwsel.hwsel_forest_pack(f)
        plain = hwsel.hwsel_forest_score(f, X, packed=packed)
        scores = torch.empty_like(plain)
        hwsel.hwsel_select_forest(hw, dp, ds, dc, F, f, packed, 3, scores=scores)
        assert torch.equal(scores, plain)


def test_many_rows_walk_whole_tiles():
    """More tiles than the split binning takes, and a matrix past the caches."""
    probs, seg, c = make(1, np.array([40_000, 1, 0, 600_003]), 2)
    dp, ds, dc = device(probs, seg, c)
    X = hwsel.hwsel_features(HW, dp, ds, dc, 128)
    rows = np.random.default_rng(2).integers(0, int(seg[-1]), 20_000)
    rows = np.unique(np.concatenate([rows, np.arange(39_900, 40_100), np.arange(int(seg[-1]) - 300, int(seg[-1]))]))
    want = oracle.features(HW, probs, seg, c, 128, rows.astype(np.int64))
    got = X[torch.from_numpy(rows).cuda()].cpu().numpy()
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    g = np.random.default_rng(3)
    T, D = 70, 6
    feat = g.integers(0, 128, (T, 63))
    thr = want[g.integers(0, 200, (T, 63)), feat].astype(np.float32)
    f = dict(n_trees=T, depth=D, n_features=128, flags=0, base_score=0.0, node_feature=hwsel.to_device(feat.astype(np.uint8)),
             node_threshold=hwsel.to_device(thr), leaf_value=hwsel.to_device(g.normal(0, 1, (T, 64)).astype(np.float32)))
    packed = hwsel.hwsel_forest_pack(f)
    scores = torch.empty(int(seg[-1]), device="cuda")
    hwsel.hwsel_select_forest(HW, dp, ds, dc, 128, f, packed, 3, scores=scores)
    assert torch.equal(scores, hwsel.hwsel_forest_score(f, X, packed=packed))


@pytest.mark.parametrize("F", [64, 96, 128])
@pytest.mark.parametrize("big", [0, 3], ids=["plain", "wide rows"])
def test_short_segments_beside_long_ones(F, big):
    """More problems in a workgroup's rows than have their terms in LDS, where
    the segments are long on average and whole tiles are walked."""
    lens = np.array([1] * 500 + [0] * 70 + [40_000] + [3] * 300 + [0, 9, 0, 64] * 5)
    probs, seg, c = make(F + big, lens, big)
    R = int(seg[-1])
    assert R >= 4 * len(lens) and R > 64 * 512
    say(f"{R} rows, F={F}")
    dp, ds, dc = device(probs, seg, c)
    X = hwsel.hwsel_features(HW, dp, ds, dc, F)
    rows = np.concatenate([np.arange(900), np.arange(39_000, R)]).astype(np.int64)
    want = oracle.features(HW, probs, seg, c, F, rows)
    assert np.array_equal(X[torch.from_numpy(rows).cuda()].cpu().numpy().view(np.uint32), want.view(np.uint32))
    g = np.random.default_rng(4)
    for nf in (F, F - 21):
        feat = g.integers(0, nf, (40, 31))
        thr = want[g.integers(0, len(want), (40, 31)), feat].astype(np.float32)
        f = dict(n_trees=40, depth=5, n_features=nf, flags=0, base_score=0.0, node_feature=hwsel.to_device(feat.astype(np.uint8)),
                 node_threshold=hwsel.to_device(thr), leaf_value=hwsel.to_device(g.normal(0, 1, (40, 32)).astype(np.float32)))
        packed = hwsel.hwsel_forest_pack(f)
        scores = torch.empty(R, device="cuda")
        hwsel.hwsel_select_forest(HW, dp, ds, dc, F, f, packed, 3, scores=scores)
        assert torch.equal(scores, hwsel.hwsel_forest_score(f, X, packed=packed))
