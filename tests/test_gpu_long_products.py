"""Products on 256x256 bf16 tiles with long contractions, against float64 on the tensors as the library stored them: forward, data gradient
and weight gradient, both layouts of the outputs and the mask bits between them.  They run on 4 wavefronts a tile from K = 3072 on where the tiles fill their last
round of 256 compute units (240 and 256 tiles here), from 4096 (forward) and 6144 (data gradient) on where they do not (272 to 425), on 8 below.

Tolerances against max|ref| of each tensor: bf16 rounds every stored tensor to 2^-9 of itself, a handful of them in a row: 2e-2.  The mask
is exact: a data gradient is zero wherever the stored activation is.  A weight gradient of stored bf16 tensors is a float32 sum of exact
products: 1e-4 is sqrt(K) 2^-24 of the row norm for K = 4352, times 25."""

import math

import pytest
import torch

from paper_2403_11204_amd import api

pytestmark = pytest.mark.gpu


def close(got, ref, tol):
    got, ref = got.double(), ref.double()
    return float((got - ref).abs().max()) <= tol * max(float(ref.abs().max()), 1e-30)


# rows and columns on, one beside and half a tile beside an edge of the 256-wide tiles; contractions of whole k-tiles of 64, of one chunk of 8
# more and of one chunk less, down to the shortest on this path; a batch shorter than what the one before it left in the buffers
@pytest.mark.parametrize("B,widths", [(4096, (3072, 4096, 4096)), (4090, (3073, 4100, 4103)), (4225, (3080, 3968, 4352)), (3841, (3135, 4097, 4031)),
                                      (4090, (3585, 4090, 4095)), (3970, (3591, 4031, 4094)), (4100, (4104, 4100, 6150))])
def test_step_against_float64(B, widths):
    g = torch.Generator(device="cuda").manual_seed(B + sum(widths))
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    seg = api.Segment(list(widths), api.RELU_ALL, api.MSE_SIL, max_batch=B + 130, dtype=api.BF16, lr=0.0, momentum=0.0)
    params = [(rand(n, k) / math.sqrt(k), rand(n) / math.sqrt(k)) for k, n in zip(widths, widths[1:])]
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    for rows in (B + 130, B):
        X, dA = rand(rows, widths[0]).bfloat16(), rand(rows, widths[-1]).bfloat16()
        seg.step_external(X, dA)
        a1, a2 = (seg.get_activation(l, rows) for l in (1, 2))
        W16 = [W.bfloat16().double() for W, _ in params]
        assert close(a1, torch.relu(X.double() @ W16[0].t() + params[0][1].double()), 2e-2)
        assert close(a2, torch.relu(a1.double() @ W16[1].t() + params[1][1].double()), 2e-2)
        dZ2, dZ1 = (seg.get_activation(l, rows, kind=1) for l in (2, 1))
        assert torch.all(dZ1[a1 <= 0] == 0)
        assert close(dZ1, (dZ2.double() @ W16[1]) * (a1 > 0), 2e-2)
        assert close(seg.get_grads(1)[0], dZ2.double().t() @ a1.double(), 1e-4)      # reads both transposed copies
        assert close(seg.get_grads(0)[0], dZ1.double().t() @ X.double(), 1e-4)


# the input gradient has no mask, the last layer of a regression no ReLU
def test_input_gradient_and_identity_output():
    B, widths = 4090, (3585, 4090, 4095)
    g = torch.Generator(device="cuda").manual_seed(11)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    seg = api.Segment(list(widths), api.RELU_HIDDEN_IDENTITY_LAST, api.MSE_SIL, max_batch=B, dtype=api.BF16, lr=0.0, momentum=0.0, input_grad=True)
    params = [(rand(n, k) / math.sqrt(k), rand(n) / math.sqrt(k)) for k, n in zip(widths, widths[1:])]
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    seg.set_labels(rand(3, widths[-1]))
    X, y = rand(B, widths[0]).bfloat16(), torch.randint(0, 3, (B,), generator=g, device="cuda", dtype=torch.int32)
    dX, _ = seg.input_grad(X, y)
    W16 = [W.bfloat16().double() for W, _ in params]
    a1, a2 = (seg.get_activation(l, B) for l in (1, 2))
    dZ2, dZ1 = (seg.get_activation(l, B, kind=1).double() for l in (2, 1))
    assert close(a2, a1.double() @ W16[1].t() + params[1][1].double(), 2e-2) and float(a2.min()) < 0
    assert close(dZ1, (dZ2 @ W16[1]) * (a1 > 0), 2e-2)
    assert close(dX, dZ1 @ W16[0], 2e-2) and torch.any(dX[X < 0] != 0)
    assert torch.equal(seg.forward(X), a2)


# the caller's own dense rows as operand and output, with rows behind them that stay as they are
@pytest.mark.parametrize("B,widths", [(4090, (3080, 4088, 3976)), (4100, (4104, 4104, 4120))])
def test_forward_into_dense_rows(B, widths):
    g = torch.Generator(device="cuda").manual_seed(12)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    seg = api.Segment(list(widths), api.RELU_HIDDEN_IDENTITY_LAST, api.MSE_SIL, max_batch=B, dtype=api.BF16, lr=0.0, momentum=0.0)
    params = [(rand(n, k) / math.sqrt(k), rand(n) / math.sqrt(k)) for k, n in zip(widths, widths[1:])]
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    X = torch.full((B + 9, widths[0]), float("nan"), device="cuda", dtype=torch.bfloat16)
    X[:B] = rand(B, widths[0])
    out = torch.full((B + 9, widths[-1]), 7.0, device="cuda", dtype=torch.bfloat16)
    seg.forward(X[:B], out=out[:B])
    W16 = [W.bfloat16().double() for W, _ in params]
    a1 = torch.relu(X[:B].double() @ W16[0].t() + params[0][1].double()).bfloat16().double()
    assert close(out[:B], a1 @ W16[1].t() + params[1][1].double(), 2e-2)
    assert torch.all(out[B:] == 7.0)


# an infinite input: its row is what IEEE arithmetic gives, and nothing of it gets into rows and columns beside the matrix
@pytest.mark.parametrize("B,widths", [(4090, (3073, 4100, 4103)), (4090, (3073, 4090, 4095))])
def test_an_infinite_input_stays_in_its_row(B, widths):
    g = torch.Generator(device="cuda").manual_seed(5)
    seg = api.Segment(list(widths), api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=api.BF16, lr=0.0, momentum=0.0)
    params = [(torch.rand((n, k), generator=g, device="cuda") / k + 1e-3, torch.zeros(n, device="cuda")) for k, n in zip(widths, widths[1:])]
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    X = torch.rand((B, widths[0]), generator=g, device="cuda").bfloat16()
    X[B - 1, 3] = float("inf")
    out = seg.forward(X)
    assert torch.all(torch.isinf(out[B - 1]))
    assert torch.all(torch.isfinite(out[: B - 1]))
    ref = torch.relu(torch.relu(X[: B - 1].double() @ params[0][0].bfloat16().double().t()) @ params[1][0].bfloat16().double().t())
    assert close(out[: B - 1], ref, 2e-2)
