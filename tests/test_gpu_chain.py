"""Forward passes of narrow layers in one launch against the same layers one handle each, which launch a product each: the same bits,
since every sum is in the same order."""

import pytest
import torch

from paper_2403_11204_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("act", [api.RELU_ALL, api.RELU_HIDDEN_IDENTITY_LAST])
# strips of 16 rows and one short, one row, more strips than compute units; widths beside the 16-byte pieces, the blocks and the k-tiles,
# a first layer that is too wide, a chain of four behind a narrow one, and rows whose start is not aligned
@pytest.mark.parametrize("B,widths", [(1, [1, 1, 1]), (16, [64, 64, 64]), (17, [32, 33, 31, 5]), (64, [60, 60, 60, 47]), (200, [784, 64, 48, 10]),
                                      (100, [15, 16, 17, 63, 64, 62]), (4096, [64, 64, 64]), (4097, [64, 40, 64, 20]), (50, [61, 20, 30])])
def test_same_bits_as_layer_by_layer(B, widths, act, dtype):
    g = torch.Generator(device="cuda").manual_seed(B + sum(widths))
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    L = len(widths) - 1
    params = [(rand(n, k) / k ** 0.5, rand(n)) for k, n in zip(widths, widths[1:])]
    seg = api.Segment(widths, act, api.MSE_SIL, max_batch=B, dtype=dtype)
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    X = rand(B, widths[0]).to(tdt)
    ref = [X]
    for l, (W, b) in enumerate(params):
        one = api.Segment(widths[l:l + 2], api.RELU_ALL if l + 1 < L else act, api.MSE_SIL, max_batch=B, dtype=dtype)
        one.set_params(0, W, b)
        ref.append(one.forward(ref[-1]))
    pad = torch.full((B * widths[-1] + 9,), 7.0, dtype=tdt, device="cuda")
    for first in (0, 1):                       # an aligned output and one that is not
        out = pad[first:first + B * widths[-1]].view(B, widths[-1])
        assert torch.equal(seg.forward(X, out=out), ref[-1])
        assert torch.all(pad[first + B * widths[-1]:] == 7.0)
    for l in range(1, L):
        assert torch.equal(seg.get_activation(l, B), ref[l])
    # an output on top of the input, as far as it fits
    if widths[-1] <= widths[0]:
        both = X.clone().view(-1)
        assert torch.equal(seg.forward(both.view(B, -1), out=both[:B * widths[-1]].view(B, widths[-1])), ref[-1])
    # a training step behind it reads its own input
    seg.step_external(X, torch.zeros_like(ref[-1]))
    assert torch.equal(seg.get_activation(0, B), X)
