"""Products of small layers against float64, at sizes on and beside the edges of their tiles (16, 32, 64) and of the rule
that picks between them.

Tolerances, against max|ref| of each tensor: float32 sums of K terms in any order are within K 2^-24 of the absolute sums,
8e-6 at the largest K here with terms of one sign, far less with both: 1e-5.  bf16 rounds every stored tensor to 2^-9 of
itself, a handful of them in a row: 2e-2 (the suite's figures)."""

import math

import pytest
import torch

from paper_2403_11204_amd import api

pytestmark = pytest.mark.gpu
TOL = {api.F32: 1e-5, api.BF16: 2e-2}
# batch, fan-in, fan-out
SHAPES = [(1, 1, 1), (15, 17, 16), (16, 128, 16), (17, 33, 47), (31, 784, 33), (64, 130, 65), (257, 64, 1000), (1410, 80, 60),
          (128, 1000, 784), (352, 96, 361), (512, 130, 1024), (1000, 300, 520), (3, 2048, 2050)]


def close(got, ref, tol):
    got, ref = got.double().cpu(), ref.cpu()
    return float((got - ref).abs().max()) <= tol * float(ref.abs().max())


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("B,K,N", SHAPES)
def test_products_of_one_layer(B, K, N, fused, dtype):
    g = torch.Generator().manual_seed(B * 7 + K * 3 + N)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    W = (torch.rand(N, K, generator=g) * 2 - 1) / math.sqrt(K)
    b = (torch.rand(N, generator=g) * 2 - 1) / math.sqrt(K)
    X = torch.rand(B, K, generator=g).to(tdt)
    y = torch.randint(0, N, (B,), generator=g, dtype=torch.int32)
    # A step moves a sample's logits by at most lr |x|^2 max P, x in [0, 1]: with lr = 1 / K by less than 1.  Larger steps
    # saturate the softmax at large K (a shift of 22 at lr = 0.1, K = 2048), and a probability of 1e-10 carries the absolute
    # rounding error of a logit of 22, 2^-24 * 22 * sqrt(K), as its relative one: 6e-5, which says nothing of the products.
    lr, mu = 1.0 / K, 0.9
    seg = api.Segment([K, N], api.RELU_HIDDEN_IDENTITY_LAST, api.SOFTMAX_XENT, max_batch=B + 3, dtype=dtype, lr=lr, momentum=mu,
                      input_grad=True)
    seg.set_params(0, W.cuda(), b.cuda())
    seg.set_fused_update(fused)
    Wop = W.to(tdt).double()                       # what the products read
    Z = X.double() @ Wop.t() + b.double()
    P = torch.softmax(Z, 1)
    P[torch.arange(B), y.long()] -= 1.0
    P /= B
    Xd, yd = X.cuda(), y.cuda()
    assert close(seg.forward(Xd), Z, TOL[dtype])
    dX, _ = seg.input_grad(Xd, yd)
    assert close(dX, P @ Wop, TOL[dtype])
    seg.step(Xd, yd)
    dW = P.t() @ X.double()
    assert close(seg.get_momentum(0)[0], dW, TOL[dtype])
    if not fused:
        assert close(seg.get_grads(0)[0], dW, TOL[dtype])
    assert close(seg.get_params(0)[0] - W.cuda(), -lr * dW, 2 * TOL[dtype] if dtype == api.BF16 else 1e-3)   # float32 masters: 2^-24 of W
    assert close(seg.get_bias_grad(0), P.sum(0), TOL[dtype])
    # the copies the products read were rewritten with the weights: the forward pass sees the new ones
    W2, b2 = seg.get_params(0)
    Z2 = X.double() @ W2.cpu().to(tdt).double().t() + b2.cpu().double()
    assert close(seg.forward(Xd), Z2, TOL[dtype])
    dX2, _ = seg.input_grad(Xd, yd)
    P2 = torch.softmax(Z2, 1)
    P2[torch.arange(B), y.long()] -= 1.0
    assert close(dX2, (P2 / B) @ W2.cpu().to(tdt).double(), TOL[dtype])


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("w0", [24, 60, 61, 64])
@pytest.mark.parametrize("wl", [8, 12, 47])
def test_workspace_copies_of_input_and_output(w0, wl, dtype):
    """Small layers read the caller's input and write its output themselves where the rows' alignment allows it: the copies
    that slp_segment_get_activation returns are made all the same, but where the interface says that X and out are used in
    place (rows of X on 128-byte boundaries with a width that divides by 64, of out on 16-byte ones with one by 8)."""
    g = torch.Generator().manual_seed(w0 + wl)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    B = 37
    seg = api.Segment([w0, 33, wl], api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=dtype)
    seg.init(3)
    table = torch.rand(5, wl, generator=g).cuda()
    seg.set_labels(table)
    X = torch.rand(B, w0, generator=g).to(tdt).cuda()
    y = torch.randint(0, 5, (B,), generator=g, dtype=torch.int32).cuda()
    out = seg.forward(X)
    if w0 != 64:
        assert torch.equal(seg.get_activation(0, B), X)
    if wl != 8:
        assert torch.equal(seg.get_activation(2, B), out)
    loss = seg.step(X, y)
    assert torch.equal(seg.get_activation(0, B), X) and torch.equal(seg.get_activation(2, B), out)
    diff = out.double() - table.double()[y.long()]
    assert abs(float(loss) - float(diff.square().mean())) <= 1e-5 * float(diff.square().mean())
    dz = torch.where(out > 0, diff * (2.0 / (B * wl)), torch.zeros_like(diff))
    assert close(seg.get_activation(2, B, kind=1), dz, TOL[dtype])
