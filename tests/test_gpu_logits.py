"""The last layer's product and the cross-entropy in one launch (up to 64 classes): edges of its 16-row strips, its 16-column tiles, its k-tiles and
its line, against float64 on the activations as the library stored them.

Tolerances against max|ref| of each tensor: 1e-5 float32 (sums of at most 1536 terms: sqrt(K) 2^-24 of the row norm is 2e-6), 2e-2 bf16
(2^-9 of each stored tensor).  The loss is a mean of float32 row losses of logits as stored: 1e-5 in both."""

import math

import pytest
import torch

from paper_2403_11204_amd import api

pytestmark = pytest.mark.gpu


def close(got, ref, tol):
    got, ref = got.double(), ref.double()
    return float((got - ref).abs().max()) <= tol * max(float(ref.abs().max()), 1e-30)


@pytest.mark.parametrize("act", [api.RELU_HIDDEN_IDENTITY_LAST, api.RELU_ALL])
@pytest.mark.parametrize("dtype,K,C", [(api.F32, 8, 1), (api.F32, 60, 47), (api.F32, 513, 17), (api.F32, 512, 48), (api.F32, 1536, 16), (api.F32, 384, 64),
                                       (api.F32, 385, 64), (api.BF16, 8, 1), (api.BF16, 60, 47), (api.BF16, 1001, 16), (api.BF16, 257, 33),
                                       (api.BF16, 4096, 64), (api.BF16, 4097, 47), (api.BF16, 300, 65),
                                       (api.F32, 1537, 16), (api.F32, 576, 32), (api.F32, 256, 33), (api.F32, 144, 49), (api.F32, 145, 64),
                                       (api.BF16, 1024, 64), (api.BF16, 1025, 49), (api.BF16, 4096, 47)])
@pytest.mark.parametrize("B", [1, 9, 16, 250])
def test_step_against_float64(dtype, K, C, act, B):
    tdt, tol = (torch.float32, 1e-5) if dtype == api.F32 else (torch.bfloat16, 2e-2)
    widths = [24, K, C]
    g = torch.Generator(device="cuda").manual_seed(B + sum(widths))
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    seg = api.Segment(widths, act, api.SOFTMAX_XENT, max_batch=B + 40, dtype=dtype, lr=0.0, momentum=0.0, input_grad=True)
    params = [(rand(n, k) / math.sqrt(k), rand(n)) for k, n in zip(widths, widths[1:])]
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    for rows in (B + 40, B):               # the second batch is shorter: what the first one left behind it is not read
        X, y = rand(rows, 24).to(tdt), torch.randint(0, C, (rows,), generator=g, device="cuda", dtype=torch.int32)
        y[0] = C                           # out of range: clamped and counted
        loss = seg.step(X, y).clone()
        a1, z = (seg.get_activation(l, rows).double() for l in (1, 2))
        pre = a1 @ params[1][0].to(tdt).double().t() + params[1][1].double()
        assert close(z, torch.relu(pre) if act == api.RELU_ALL else pre, tol)
        ids = y.long().clamp(max=C - 1)
        lse = torch.logsumexp(z, 1)
        ref = torch.exp(z - lse[:, None])
        ref[torch.arange(rows), ids] -= 1.0
        ref /= rows
        if act == api.RELU_ALL:
            ref *= z > 0
        dZ = seg.get_activation(2, rows, kind=1).double()
        assert float((dZ - ref).abs().max()) <= tol / rows          # softmax and one-hot are at most 1
        expected = (lse - z.gather(1, ids[:, None])[:, 0]).mean()
        assert abs(float(loss) - float(expected)) <= 1e-5 * max(1.0, abs(float(expected)))
        dW, db = seg.get_grads(1)                                     # read the transposed gradient
        scale = float((dZ.abs().t() @ a1.abs()).max()) + 1e-30
        assert float((dW.double() - dZ.t() @ a1).abs().max()) <= 1e-5 * scale
        assert float((db.double() - dZ.sum(0)).abs().max()) <= 1e-5 * float(dZ.abs().sum(0).max() + 1e-30)
        dX, loss2 = seg.input_grad(X, y)                              # the same without the transposed gradient
        assert torch.equal(loss2, loss)
        assert torch.equal(seg.get_activation(2, rows, kind=1).double(), dZ)
    assert seg.target_errors() == 4


# a gradient from outside on a segment of this kind does not take the cross-entropy's way
def test_external_gradient_on_a_classifier():
    widths, rows = [24, 60, 47], 50
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    seg = api.Segment(widths, api.RELU_HIDDEN_IDENTITY_LAST, api.SOFTMAX_XENT, max_batch=rows, lr=0.0, momentum=0.0)
    for l, (k, n) in enumerate(zip(widths, widths[1:])):
        seg.set_params(l, rand(n, k), rand(n))
    dA = rand(rows, 47)
    seg.step_external(rand(rows, 24), dA)
    assert torch.equal(seg.get_activation(2, rows, kind=1), dA)
    assert seg.target_errors() == 0


# the launch gives the bits of the two it takes the place of: hidden units that are always zero change no sum, but take a layer over the line to them;
# and the logits are those of the forward-only pass
@pytest.mark.parametrize("dtype,K,beyond,C", [(api.F32, 1536, 1544, 16), (api.F32, 570, 584, 30), (api.F32, 255, 272, 47), (api.F32, 144, 160, 64),
                                              (api.BF16, 1000, 1032, 64), (api.BF16, 4096, 4104, 47)])
@pytest.mark.parametrize("act", [api.RELU_HIDDEN_IDENTITY_LAST, api.RELU_ALL])
@pytest.mark.parametrize("B", [3, 130])
def test_same_bits_as_product_and_cross_entropy_apart(dtype, K, beyond, C, act, B):
    g = torch.Generator(device="cuda").manual_seed(K + C + B)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    W1, b1, W2, b2 = rand(K, 24), rand(K), rand(C, K) / math.sqrt(K), rand(C)
    X, y = rand(B, 24).to(torch.float32 if dtype == api.F32 else torch.bfloat16), torch.randint(0, C, (B,), generator=g, device="cuda", dtype=torch.int32)
    outs = []
    for k in (K, beyond):
        seg = api.Segment([24, k, C], act, api.SOFTMAX_XENT, max_batch=B, dtype=dtype, lr=0.0, momentum=0.0)
        seg.set_params(0, torch.cat([W1, W1.new_zeros(k - K, 24)]), torch.cat([b1, b1.new_zeros(k - K)]))
        seg.set_params(1, torch.cat([W2, W2.new_zeros(C, k - K)], 1), b2)
        loss = seg.step(X, y).clone()
        z = seg.get_activation(2, B)
        assert torch.equal(z, seg.forward(X))
        dW, db = seg.get_grads(1)
        outs.append((loss, z, seg.get_activation(2, B, kind=1), dW[:, :K].clone(), db))
    for one, two in zip(*outs):
        assert torch.equal(one, two)
