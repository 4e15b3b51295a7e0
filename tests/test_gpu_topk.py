"""Top-k where its bound can go wrong: score orders that put the best rows in
one lane, one wave or the last tile, more equal or rising scores than its list
holds, NaN, lengths around a tile, few problems (large workgroups) and many."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


def orders(g, n):
    i = np.arange(n)
    base = g.standard_normal(n).astype(np.float32)
    yield "random", base
    yield "rising", i.astype(np.float32)
    yield "falling", -i.astype(np.float32)
    yield "equal", np.full(n, 2.5, np.float32)
    yield "few levels", g.integers(0, 3, n).astype(np.float32)
    yield "one lane of 1,024", np.where(i % 1024 == 77, base + 100, base).astype(np.float32)
    yield "one lane of 256", np.where(i % 256 == 200, base + 100, base).astype(np.float32)
    yield "one wave", np.where(i % 256 < 64, base + 100, base).astype(np.float32)
    yield "nan", np.where(g.random(n) < 0.9, np.nan, base).astype(np.float32)
    yield "all nan", np.full(n, np.nan, np.float32)
    yield "tiles rise", (i // 8192 * 10 + base).astype(np.float32)


@pytest.mark.parametrize("many", [False, True], ids=["few problems", "many problems"])
@pytest.mark.parametrize("k", [1, 7, 16, 33, 64])
def test_topk_orders(k, many):
    g = np.random.default_rng(k)
    parts = [s for n in (1, 63, 513, 8191, 8192, 8193, 20_000) for _, s in orders(g, n)]
    if many:                                                    # past 256 problems: small workgroups
        parts += [g.standard_normal(int(n)).astype(np.float32) for n in g.integers(0, 40, 300)]
    say(f"k={k}: {len(parts)} segments")
    seg = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
    s = np.concatenate(parts)
    idx, vals = hwsel.hwsel_topk_per_problem(torch.from_numpy(s).cuda(), torch.from_numpy(seg).cuda(), k)
    oidx, ovals = oracle.topk(s, seg, k)
    bad = np.argwhere((idx.cpu().numpy() != oidx).any(1)).ravel()
    assert len(bad) == 0, f"segments {bad[:5]}"
    assert np.array_equal(vals.cpu().numpy().view(np.uint32), ovals.view(np.uint32))
    rt = np.abs(s)
    r = hwsel.hwsel_regret(torch.from_numpy(rt).cuda(), torch.from_numpy(seg).cuda(), idx)
    for got, want in zip(r, oracle.regret(rt, seg, oidx)):
        assert np.array_equal(got.cpu().numpy(), want, equal_nan=got.dtype == torch.float32)


# by length: one wave up to 64 rows, 256 threads up to 1,024, tiles beyond
@pytest.mark.parametrize("many", [False, True], ids=["few problems", "many problems"])
@pytest.mark.parametrize("k", [1, 5, 64])
def test_topk_short_segments(k, many):
    g = np.random.default_rng(100 + k)
    lens = [0, 1, 2, 4, 63, 64, 65, 127, 255, 256, 257, 512, 513, 1023, 1024, 1025] * (17 if many else 1)
    parts = [s for n in set(lens) if n for _, s in orders(g, n)] if not many else []
    parts += [g.standard_normal(n).astype(np.float32) for n in lens]
    seg = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
    s = np.concatenate(parts)
    say(f"k={k}: {len(parts)} segments")
    idx, vals = hwsel.hwsel_topk_per_problem(torch.from_numpy(s).cuda(), torch.from_numpy(seg).cuda(), k)
    oidx, ovals = oracle.topk(s, seg, k)
    assert np.array_equal(idx.cpu().numpy(), oidx)
    assert np.array_equal(vals.cpu().numpy().view(np.uint32), ovals.view(np.uint32))
    rt = np.abs(s)
    r = hwsel.hwsel_regret(torch.from_numpy(rt).cuda(), torch.from_numpy(seg).cuda(), idx)
    for got, want in zip(r, oracle.regret(rt, seg, oidx)):
        assert np.array_equal(got.cpu().numpy(), want, equal_nan=got.dtype == torch.float32)
