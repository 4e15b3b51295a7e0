"""More problems than one launch of a workgroup each can hold (2^32 threads):
every problem has its own result."""
import pytest
import torch

from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [(1 << 21) + 3, (1 << 23) + 9, (1 << 24) + 1])
def test_two_rows_a_problem(P):
    say(f"{P} problems")
    g = torch.Generator(device="cuda").manual_seed(P)
    t = 1 + torch.rand(P, 2, generator=g, device="cuda")
    seg = 2 * torch.arange(P + 1, device="cuda")
    slow, fast = (t[:, 1] > t[:, 0]).int(), (t[:, 1] < t[:, 0]).int()          # the first of two equal ones
    want = 1 - t.min(1).values.double() / t.max(1).values.double()
    idx, vals = hwsel.hwsel_topk_per_problem(t.view(-1), seg, 1)
    assert torch.equal(idx.view(-1), slow) and torch.equal(vals.view(-1), t.max(1).values)
    r1, rk, best = hwsel.hwsel_regret(t.view(-1), seg, idx)
    assert torch.equal(r1, want.float()) and torch.equal(rk, r1) and torch.equal(best, fast)
    # the id of the second row is 1, where it is the faster 64: one y each
    ids = torch.stack([torch.zeros_like(fast), torch.where(fast == 1, 64, 1).int()], 1).view(-1)
    (id_, count), mean = (v.cpu() for v in hwsel.hwsel_static_config(t.view(-1), seg, ids, 65))
    y0 = torch.where(fast == 0, torch.ones_like(want), 1 - want)
    # P fp64 additions in order are within P 2^-53 of their sum
    assert int(id_) == 0 and int(count) == P and abs(float(mean[0]) - float(y0.mean())) < 2 * P * 2.0 ** -53
    if P > 1 << 23:
        return                                     # (the aggregates add problem after problem: over a second)
    out, reg, rank, ybar = hwsel.hwsel_evaluate(t.view(-1), seg, idx)
    assert float(out[8]) == P and torch.equal(rank, 1 + (t[:, 0] != t[:, 1]).int())
    assert torch.equal(reg, 1 - t.min(1).values.double() / t.max(1).values.double())
    assert torch.equal(ybar, (1 + t.min(1).values.double() / t.max(1).values.double()) / 2)


def test_evaluate_many():
    P = (1 << 23) + 9
    say(f"evaluate {P} problems")
    t = torch.tensor([1.0, 2.0], device="cuda").repeat(P)
    seg = 2 * torch.arange(P + 1, device="cuda")
    idx = (torch.arange(P, device="cuda") % 2).int().view(P, 1)
    out, reg, rank, ybar = hwsel.hwsel_evaluate(t, seg, idx)
    assert torch.equal(reg, 0.5 * idx.view(-1).double()) and torch.equal(rank, 1 + idx.view(-1))
    assert bool((ybar == 0.75).all()) and float(out[8]) == P and float(out[3]) == 0.5
