"""Selection metrics and the static baseline where their dispatch and tiling
can go wrong: problem counts around a wave and a step, regrets of which many
or all are equal, rows grouped by id ranges or kept as a table, ids in any
order, repeated, out of range.  Against the oracle; every value is
exact but the means of y (fp64 sums in another order)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


def up(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("P", [1, 2, 63, 64, 65, 255, 257, 1025, 4096, 4097])
@pytest.mark.parametrize("kind", ["spread", "zeros", "few", "equal"])
def test_order_statistics(P, kind):
    """Two rows a problem, the pick the slower by a factor that fixes the regret."""
    say(f"evaluate {P} problems, {kind}")
    g = np.random.default_rng(P)
    slow = {"spread": 1 + g.random(P), "zeros": np.where(g.random(P) < 0.7, 1, 1 + g.random(P)),
            "few": 1 + g.integers(0, 3, P), "equal": np.full(P, 1.5)}[kind]
    rt = np.stack([np.ones(P), slow], 1).astype(np.float32).ravel()
    seg = 2 * np.arange(P + 1, dtype=np.int64)
    idx = np.where(g.random((P, 1)) < 0.1, -1, 1).astype(np.int32)
    agg, reg, rank, ybar = oracle.evaluate(rt, seg, idx)
    out, *got = (t.cpu().numpy() for t in hwsel.hwsel_evaluate(up(rt), up(seg), up(idx)))
    for a, b in zip(got, (reg, rank, ybar)):
        assert np.array_equal(a, b, equal_nan=True)
    want = np.array([agg[f] for f in oracle.EVAL_FIELDS])
    assert np.array_equal(out, want, equal_nan=True), (out, want)


@pytest.mark.parametrize("P,n_cfg", [(1, 1), (1, 64), (3, 65), (8, 4097), (9, 1001), (127, 640), (129, 6401),
                                     (5, 655_360), (5, 655_361)])
@pytest.mark.parametrize("order", ["sorted", "shuffled", "repeated"])
def test_static_config(P, n_cfg, order):
    """Segments from empty to twice as long as there are ids: with many rows
    per id a call keeps them as a table, with few it groups them."""
    say(f"static config {P} problems, {n_cfg} ids, {order}")
    g = np.random.default_rng(P * n_cfg)
    ids, lens = [], []
    for p in range(P):
        if order == "repeated":
            i = g.integers(-2, n_cfg + 2, int(g.choice([0, 1, 63, 700, min(2 * n_cfg, 9000)])))
        else:
            share = 1 if n_cfg < 4000 and p % 3 else (0.45, 0.9)[p % 2]
            i = np.flatnonzero(g.random(n_cfg) < share)
            if order == "shuffled":
                g.shuffle(i)
        ids.append(i)
        lens.append(len(i))
    check_static(g, ids, lens, n_cfg)


def check_static(g, ids, lens, n_cfg):
    ids = np.concatenate(list(ids) + [np.zeros(1)]).astype(np.int32)      # a row past the last segment is no one's
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rt = g.lognormal(0, 0.3, len(ids)).astype(np.float32)
    rt[g.random(len(rt)) < 0.05] = np.inf
    rt[g.random(len(rt)) < 0.02] = np.nan
    best, mean = hwsel.hwsel_static_config(up(rt), up(seg), up(ids), n_cfg)
    ob, oc, oy = oracle.static_config(rt, seg, ids, n_cfg)
    assert (int(best[0]), int(best[1])) == (ob, oc)
    assert np.array_equal(mean.cpu().numpy()[0], oy, equal_nan=True)


@pytest.mark.parametrize("P,n_cfg", [(1, 4097), (9, 1001), (65, 640), (129, 3000)])
@pytest.mark.parametrize("order", ["sorted", "shuffled"])
@pytest.mark.parametrize("share", [0.02, 0.3, "fits", "too many"])
def test_static_config_grouped(P, n_cfg, order, share):
    """A share of the ids per problem, every id once: runs of rows of one range
    from one row to whole ranges, across lanes, waves and steps.  The rows are
    grouped where 2 words each fit beside every problem's range starts, the
    last two cases lie on both sides of that."""
    ranges = -(-n_cfg // 64)
    most = (P * n_cfg - (P * (ranges + 1) + 1 & ~1)) // 2            # rows that are grouped
    g = np.random.default_rng(P + n_cfg)
    total = most if share == "fits" else most + 1 if share == "too many" else int(share * P * n_cfg)
    lens = [total * (p + 1) // P - total * p // P for p in range(P)]
    assert max(lens) <= n_cfg
    say(f"static config {P} problems, {n_cfg} ids, {total} rows ({most} grouped at most), {order}")
    common = g.permutation(n_cfg)                                     # so that some ids are in most problems
    ids = []
    for n in lens:
        i = common[:n] if share != 0.02 else np.unique(np.r_[common[:n // 2], g.permutation(n_cfg)])[:n]
        i = g.permutation(i) if order == "shuffled" else np.sort(i)
        ids.append(i)
    check_static(g, ids, [len(i) for i in ids], n_cfg)
