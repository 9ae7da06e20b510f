"""Launches of one or two products on 128x128 or 64x128 tiles with the update in the epilogue, against float64: a weight gradient
alone, with the data gradient below it, two weight gradients, beside the caller's stream, and past the caches.

Reference: the activations as the library stored them (so that a unit at zero to rounding is on the same side), everything else
in float64.  Tolerances against max|ref| of each tensor, as for the products of small layers: float32 sums of K <= 2100 terms in
any order are within K 2^-24 of the absolute sums, 1e-5 with terms of both signs; bf16 rounds every stored tensor to 2^-9 of
itself, a handful of them in a row: 2e-2."""

import math

import pytest
import torch

from paper_2403_11204_amd import api

pytestmark = pytest.mark.gpu
TOL = {api.F32: 1e-5, api.BF16: 2e-2}
# batch, widths: more than 223 128x128 tiles a weight matrix (or a pair that has them together with one that 64x64 tiles took), rows and
# columns on and beside the edges of the tiles, contractions of less than one k-tile, one, and a remainder
CASES = [(1, [40, 3586, 1025]), (64, [1793, 2047]), (300, [130, 2050, 2047]), (257, [2047, 1800, 1921, 700]), (130, [784, 4096, 1024]),
         (1000, [784, 1500, 3001, 777])]
LARGE = [(192, [4096, 4096, 4100])]             # 0.6 GB of parameters: past the memory-side cache


def close(got, ref, tol):
    got, ref = got.double(), ref.double()
    return float((got - ref).abs().max()) <= tol * max(float(ref.abs().max()), 1e-30)


def run(B, widths, dtype, fused, mu, overlap):
    g = torch.Generator(device="cuda").manual_seed(B + sum(widths))
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda") * 2 - 1
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    L, lr = len(widths) - 1, 0.05
    seg = api.Segment(widths, api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=dtype, lr=lr, momentum=mu)
    params = [(rand(n, k) / math.sqrt(k), rand(n) / math.sqrt(k)) for k, n in zip(widths, widths[1:])]
    for l, (W, b) in enumerate(params):
        seg.set_params(l, W, b)
    seg.set_fused_update(fused)
    seg.set_overlap(overlap)
    vel = [(torch.zeros_like(W).double(), torch.zeros_like(b).double()) for W, b in params]
    for step in range(2):              # the second step reads the copies that the first one wrote
        X, dA = rand(B, widths[0]).to(tdt), rand(B, widths[-1]).to(tdt)
        before = [seg.get_params(l) for l in range(L)]
        seg.step_external(X, dA)
        acts = [X] + [seg.get_activation(l, B) for l in range(1, L + 1)]
        for l in range(1, L + 1):
            W, b = before[l - 1]
            assert close(acts[l], torch.relu(acts[l - 1].double() @ W.to(tdt).double().t() + b.double()), TOL[dtype]), ("A", l)
        dZ = dA.double() * (acts[L] > 0)
        for l in range(L, 0, -1):
            W, b = before[l - 1]
            assert close(seg.get_activation(l, B, kind=1), dZ, TOL[dtype]), ("dZ", l)
            dZ = seg.get_activation(l, B, kind=1).double()
            dW, db = dZ.t() @ acts[l - 1].double(), dZ.sum(0)
            vW, vb = mu * vel[l - 1][0] + dW, mu * vel[l - 1][1] + db
            if not fused:
                assert close(seg.get_grads(l - 1)[0], dW, TOL[dtype]), ("dW", l)
            assert close(seg.get_bias_grad(l - 1), db, TOL[dtype]), ("db", l)
            if mu:
                gW, gb = seg.get_momentum(l - 1)
                assert close(gW, vW, TOL[dtype]) and close(gb, vb, TOL[dtype]), ("v", l)
            W2, b2 = seg.get_params(l - 1)
            # the difference of two float32 numbers up to 2^-24 of the weights off
            slack = 2.0 ** -23 / (lr * float(vW.abs().max())) * float(W.abs().max())
            assert close(W2.double() - W.double(), -lr * vW, TOL[dtype] + slack), ("W", l)
            slack = 2.0 ** -23 / (lr * float(vb.abs().max())) * float(b.abs().max())
            assert close(b2.double() - b.double(), -lr * vb, TOL[dtype] + slack), ("b", l)
            vel[l - 1] = (vW, vb)
            if l > 1:
                dZ = (dZ @ W.to(tdt).double()) * (acts[l - 1] > 0)
    return [t for l in range(L) for t in seg.get_params(l)]


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("fused,mu,overlap", [(0, 0.9, False), (1, 0.9, False), (1, 0.0, False), (0, 0.9, True)])
@pytest.mark.parametrize("B,widths", CASES)
def test_steps_against_float64(B, widths, fused, mu, overlap, dtype):
    run(B, widths, dtype, fused, mu, overlap)


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("B,widths", LARGE)
def test_past_the_caches(B, widths, dtype):
    apart = run(B, widths, dtype, 0, 0.9, False)
    for a, b in zip(apart, run(B, widths, dtype, 1, 0.9, False)):     # the gradient stored or not: the same bits
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("B", [300, 1500])         # with overlap on in the product's launch as well, and apart: the two kernels' sums
def test_beside_the_stream_and_in_it_leave_the_same_bits(B, dtype):
    for a, b in zip(run(B, [130, 2050, 2047], dtype, 0, 0.9, False), run(B, [130, 2050, 2047], dtype, 0, 0.9, True)):
        assert torch.equal(a, b)


# a layer above the second of whole rounds of 256x256 tiles has its update apart, those below share launches; against all of them apart
def test_upper_layer_apart():
    widths = [130, 2050, 2047, 4090, 4093]
    for a, b in zip(run(1600, widths, api.BF16, 0, 0.9, False), run(1600, widths, api.BF16, 0, 0.9, True)):
        assert torch.equal(a, b)


def test_upper_layer_apart_in_replayed_steps():
    widths, B = [130, 2050, 2047, 4090, 4093], 1600
    g = torch.Generator(device="cuda").manual_seed(B)
    X = torch.rand((B, widths[0]), generator=g, device="cuda").bfloat16()
    y = torch.randint(0, 20, (B,), generator=g, device="cuda", dtype=torch.int32)
    table = torch.rand((20, widths[-1]), generator=g, device="cuda")
    stream, runs = torch.cuda.Stream(), []
    stream.wait_stream(torch.cuda.current_stream())
    for graph in (False, True):
        with torch.cuda.stream(stream):
            seg = api.Segment(widths, api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=api.BF16, lr=0.05, momentum=0.9)
            seg.init(5)
            seg.set_labels(table)
            seg.set_graph(graph)
            seen = []
            for _ in range(4):                 # eager work between the replays
                seen.append(seg.step(X, y).clone())
                seen.append(seg.forward(X))
            seen += [t for l in range(seg.L) for t in (*seg.get_params(l), *seg.get_momentum(l), *seg.get_grads(l))]
        stream.synchronize()
        assert (seg.graph_stats()[1] > 0) == graph
        runs.append(seen)
    for a, b in zip(*runs):
        assert torch.equal(a, b)
