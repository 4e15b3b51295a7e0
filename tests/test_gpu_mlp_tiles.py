"""The matrix-core MLP at the edges of its tile heights: rows of 32- and 64-row
tiles alone, full rounds of 128-row tiles with and without rows left over.  A
row's products and sums do not depend on the tile it is in, so its score is
the same bits in every call; a sample is compared with the fp32 row-block
path."""
import pytest
import torch

from paper_2609_35587_amd import hwsel
from _gpu_util import say

pytestmark = pytest.mark.gpu


def make_mlp(g):
    widths, m = (128, 512, 512, 256, 1), {}
    for l in range(4):
        fi, fo = widths[l], widths[l + 1]
        w = torch.randn(fo, fi, generator=g, device="cuda") * (2 / fi) ** 0.5
        m["W%d" % (l + 1)] = w.bfloat16().view(torch.int16)
        m["b%d" % (l + 1)] = (2 * torch.rand(fo, generator=g, device="cuda") - 1) / fi ** 0.5
    m["mean"] = torch.randn(128, generator=g, device="cuda")
    m["inv_std"] = 0.5 + torch.rand(128, generator=g, device="cuda")
    return m


@pytest.mark.parametrize("rounds", [0, 1, 2])
@pytest.mark.parametrize("left", [1, 31, 32, 33, 8191, 8192, 8193, 16383, 16384, 16385])
def test_same_bits_in_every_tile(rounds, left):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    R = 128 * n_cu * rounds + left
    say(f"mlp {R} rows")
    g = torch.Generator(device="cuda").manual_seed(R)
    m = make_mlp(g)
    packed = hwsel.hwsel_mlp_pack(m)
    ld = 128 if left % 2 else 132
    X = torch.randn(R, ld, generator=g, device="cuda")
    X[::97, 5] = float("nan")
    got = torch.full((R + 1,), 7.0, device="cuda")
    hwsel.hwsel_mlp_score(m, X, scores=got[:R], packed=packed)
    assert float(got[R]) == 7.0 and bool(torch.isfinite(got[:R]).all())
    # the last rows by themselves, in 32-row tiles, from another row of a tile
    n = min(R, 203)
    assert torch.equal(hwsel.hwsel_mlp_score(m, X[R - n:].contiguous(), packed=packed), got[R - n:R])
    # activations rounded to bf16 three times on either side, as in the parity tests
    ref = hwsel.hwsel_mlp_score(m, X[R - n:].contiguous())
    assert float((got[R - n:R] - ref).norm() / ref.norm()) < 2e-2
