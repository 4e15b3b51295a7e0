"""Compaction of catalogue masks, a problem's scan split over one to all of its
steps (by the number of problems), against the positions of the mask's set
bytes; and the mask's bytes against the oracle where its rules meet."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu
N = hwsel.HWSEL_CATALOGUE_SIZE


@pytest.mark.parametrize("P", [1, 2, 15, 16, 17, 33, 61, 171, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("share", [0.0, 0.01, 0.4, 1.0])
def test_compact(P, share):
    say(f"compact {P} problems, share {share}")
    g = torch.Generator(device="cuda").manual_seed(P)
    mask = (torch.rand(P, N, generator=g, device="cuda") < share).to(torch.uint8)
    mask[0, -1] = 1
    n = mask.sum(1, dtype=torch.int64)
    total = int(n.sum())
    seg, point = hwsel.hwsel_catalogue_compact(mask, n, total)
    assert torch.equal(seg[1:], torch.cumsum(n, 0)) and int(seg[0]) == 0
    assert torch.equal(point, mask.nonzero()[:, 1].int())
    if total > 5:                                             # a list cut short
        _, part = hwsel.hwsel_catalogue_compact(mask, n, total - 5)
        assert torch.equal(part, point[:total - 5])
