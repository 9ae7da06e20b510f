"""A batch that overflows leaves nothing behind: after slp_segment_init a handle steps to the bits of a new one.

The pads of the weights and of their copies are multiplied with the zeros that pad the other operand, so an infinity or a NaN that an
update let into them would turn every later step to NaN, also behind new weights."""

import pytest
import torch

from paper_2403_11204_amd import api

pytestmark = pytest.mark.gpu

# batch, widths, fused update: every place an update is written from.  Widths beside the pads of a transposed copy's rows (8) and of the
# columns of weights and momenta (4).
CASES = [(200, [784, 2048, 2052], 0), (64, [784, 2048, 2052], 1), (200, [784, 2052, 2049], 0),      # the update in a launch of larger products
         (200, [783, 2047, 2050], 0), (64, [130, 2050, 2047], 1),
         (50, [64, 60, 52], 0), (64, [1000, 1028, 1028], 0),                                        # small products
         (50, [45, 61, 50], 0), (33, [201, 330, 27], 1), (64, [1001, 1031, 1025], 0),
         (4100, [784, 2052, 2049], 0), (4100, [784, 2052, 2049], 1),                                # 128x128 tiles, gradient stored and not
         (4100, [785, 2050, 2047], 0), (4100, [785, 2050, 2047], 1),
         (4100, [784, 4092, 3588], 0), (4100, [784, 4092, 3588], 1),                                # 256x256
         (4100, [785, 4090, 3590], 0), (4100, [785, 4090, 3590], 1)]


def outcome(seg, X, y):
    seen = [seg.step(X, y).clone(), seg.forward(X)]
    seen.append(seg.step(X, y).clone())                # reads what the first step wrote
    return seen + [t for l in range(seg.L) for t in (*seg.get_params(l), *seg.get_momentum(l))]


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("B,widths,fused", CASES)
def test_init_after_an_overflowed_batch(B, widths, fused, bad, dtype):
    g = torch.Generator(device="cuda").manual_seed(B + sum(widths))
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    X = torch.rand((B, widths[0]), generator=g, device="cuda").to(tdt)
    y = torch.randint(0, 12, (B,), generator=g, device="cuda", dtype=torch.int32)
    table = torch.rand((12, widths[-1]), generator=g, device="cuda")
    runs = []
    for overflow in (False, True):
        seg = api.Segment(widths, api.RELU_HIDDEN_IDENTITY_LAST, api.MSE_SIL, max_batch=B, dtype=dtype, lr=0.05, momentum=0.9)
        seg.set_labels(table)
        seg.set_fused_update(fused)
        seg.init(3)
        if overflow:
            Xbad = X.clone()
            Xbad[B // 2, widths[0] // 2] = bad
            seg.step(Xbad, y)
            assert not all(torch.isfinite(seg.get_params(l)[0]).all() for l in range(2))
            seg.init(3)
        runs.append(outcome(seg, X, y))
    assert all(torch.isfinite(t.float()).all() for t in runs[0])
    for a, b in zip(*runs):
        assert torch.equal(a, b)


# chains of narrow layers, and products on 128x64, 128x128 and 256x256 tiles
@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("B,widths", [(50, [61, 20, 30]), (100, [15, 16, 17, 63, 62]), (1000, [70, 1500]), (1000, [70, 2055, 37]), (2100, [70, 6150])])
def test_rows_of_a_batch_do_not_meet(B, widths, bad, dtype):
    g = torch.Generator(device="cuda").manual_seed(B + sum(widths))
    X = torch.rand((B, widths[0]), generator=g, device="cuda").to(torch.float32 if dtype == api.F32 else torch.bfloat16)
    seg = api.Segment(widths, api.RELU_HIDDEN_IDENTITY_LAST, api.MSE_SIL, max_batch=B, dtype=dtype)
    seg.init(3)
    ref = seg.forward(X)
    row = B // 2
    X[row, -1] = bad
    got = seg.forward(X)
    if len(widths) == 2:               # (a unit that is not a number counts as zero behind a hidden layer)
        assert not torch.isfinite(got[row].float()).any()
    keep = torch.arange(B, device="cuda") != row
    assert torch.isfinite(got[keep].float()).all() and torch.equal(got[keep], ref[keep])
