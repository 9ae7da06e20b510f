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
@pytest.mark.parametrize("K", [40, 200, 784, 1023, 4096])
def test_tiles_16_and_32_leave_the_same_bits(K, dtype):
    """Elements of an output do not depend on each other, so the same ones as part of a small output (tile 16) and of a larger
    one (tile 32) differ only by the order of their sums: not at all.  K leaves one, an odd and an even number of k-tiles.  The
    weight gradient is seen in float32, the other two products as stored."""
    g = torch.Generator().manual_seed(K)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    n, big = 48, 640                    # 3 x 3 16x16 tiles; 40 x 40 of them are 10 x 10 64x64 ones: tile 32
    W1, W2 = torch.randn(big, K, generator=g), torch.randn(K, big, generator=g)
    X = torch.randn(big, K, generator=g).to(tdt).cuda()
    XT, dAT = torch.randn(K, big, generator=g).to(tdt).cuda(), torch.randn(K, big, generator=g).to(tdt).cuda()
    dA = torch.randn(big, K, generator=g).to(tdt).cuda()
    outs = []
    for m in (n, big):
        def segment(widths, batch):
            return api.Segment(widths, api.RELU_HIDDEN_IDENTITY_LAST, api.SOFTMAX_XENT, max_batch=batch, dtype=dtype, lr=0.0, momentum=0.5)

        fwd = segment([K, m], m)
        fwd.set_params(0, W1[:m].cuda(), torch.zeros(m).cuda())
        wgrad = segment([m, m], K)      # contraction over a batch of K rows
        wgrad.init(1)
        wgrad.step_external(XT[:, :m].contiguous(), dAT[:, :m].contiguous())
        dgrad = segment([8, m, K], m)   # hidden units all at one, so that the mask passes every element
        dgrad.set_params(0, torch.zeros(m, 8).cuda(), torch.ones(m).cuda())
        dgrad.set_params(1, W2[:, :m].contiguous().cuda(), torch.zeros(K).cuda())
        dgrad.step_external(torch.zeros(m, 8, dtype=tdt, device="cuda"), dA[:m].contiguous())
        outs.append([t[:n, :n] for t in (fwd.forward(X[:m]), wgrad.get_momentum(0)[0], dgrad.get_activation(1, m, kind=1))])
    for a, b in zip(*outs):
        assert torch.count_nonzero(a) > 0.9 * a.numel() and torch.equal(a, b)


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


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("shift", [0, 1, -1])
@pytest.mark.parametrize("B,widths", [(70, [80, 80]), (70, [61, 61]), (300, [64, 64]), (200, [1024, 1024]), (1000, [1600, 1500]), (70, [80, 40, 96])])
def test_forward_into_its_own_input(B, widths, shift, dtype):
    """out on X itself, or some rows before or behind: one layer's only launch reads the one and writes the other, at widths
    that it could take from X as they are (80; 64, 1024 and 1600 with rows on cache lines) and one that it could not (61).
    The same bits as into a buffer of its own."""
    g = torch.Generator().manual_seed(B + widths[0])
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    seg = api.Segment(widths, api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=dtype)
    seg.init(3)
    X = torch.rand(B, widths[0], generator=g).to(tdt).cuda()
    ref = seg.forward(X).clone()
    most, far = B * max(widths), shift * (B // 3) * 64             # elements; whole cache lines
    buf = torch.zeros(most + 2 * abs(far) + 64, dtype=tdt, device="cuda")
    x0 = abs(far) + 64 // buf.element_size() if widths[0] == 80 else abs(far)
    xin = buf[x0:x0 + B * widths[0]].view(B, widths[0])
    out = buf[x0 + far:x0 + far + B * widths[-1]].view(B, widths[-1])
    xin.copy_(X)
    assert torch.equal(seg.forward(xin, out=out), ref)


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("B,K,N", [(1000, 1500, 1490), (1030, 200, 2300), (1500, 200, 3500), (4090, 100, 500)])
def test_products_on_the_tiles_between_small_and_large(B, K, N, dtype):
    """bf16: 128x64 tiles (1000 x 1490, 4090 x 500), 128x128 on part of the chip (1030 x 2300), two workgroups per unit (1500 x
    3500)."""
    test_products_of_one_layer(B, K, N, 0, dtype)


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("B,C", [(1, 1), (3, 2), (5, 63), (8, 64), (13, 65), (40, 128), (21, 129), (66, 256), (31, 257), (129, 1000)])
def test_cross_entropy_gradient_and_its_transpose(B, C, dtype):
    """Classes on and beside the sizes that stay in registers (64, 128 in bf16, 256 in float32), batches that leave a wavefront's four rows and the
    padded columns of the transposed gradient partly filled: dZ, its column sums (read from the transpose) and the loss."""
    g = torch.Generator().manual_seed(B * 1000 + C)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    K = 24
    seg = api.Segment([K, C], api.RELU_HIDDEN_IDENTITY_LAST, api.SOFTMAX_XENT, max_batch=B, dtype=dtype, lr=0.0, momentum=0.0)
    W, b = torch.randn(C, K, generator=g), torch.randn(C, generator=g)
    seg.set_params(0, W.cuda(), b.cuda())
    X = torch.rand(B, K, generator=g).to(tdt)
    y = torch.randint(0, C, (B,), generator=g, dtype=torch.int32)
    loss = float(seg.step(X.cuda(), y.cuda()))
    Z = seg.get_activation(1, B).cpu().double()       # the stored logits are what the loss reads
    lse = torch.logsumexp(Z, 1)
    ref = float((lse - Z[torch.arange(B), y.long()]).mean())
    # float32: the log-sum and a logit of up to 10 each carry 2^-24 of themselves, absolutely
    assert abs(loss - ref) <= 1e-5 * max(abs(ref), 1.0)
    P = torch.exp(Z - lse[:, None])
    P[torch.arange(B), y.long()] -= 1.0
    P /= B
    scale = max(float(P.abs().max()), 1e-6 / B)       # one class: the gradient is zero to rounding
    assert float((seg.get_activation(1, B, kind=1).cpu().double() - P).abs().max()) <= TOL[dtype] * scale + 1e-6 / B
    assert float((seg.get_bias_grad(0).cpu().double() - P.sum(0)).abs().max()) <= TOL[dtype] * scale * math.sqrt(B) + 1e-6
    assert float((seg.get_grads(0)[0].cpu().double() - P.t() @ X.double()).abs().max()) <= TOL[dtype] * scale * math.sqrt(B) + 1e-6


@pytest.mark.parametrize("relu", [api.RELU_ALL, api.RELU_HIDDEN_IDENTITY_LAST])
@pytest.mark.parametrize("external", [False, True])
@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("B,N", [(5, 3), (37, 61), (64, 64), (333, 513), (330, 512), (1000, 777), (1001, 776)])
def test_gradient_of_the_output_formed_by_the_last_product(B, N, dtype, external, relu):
    """Squared error against the label table or the caller's gradient, in the epilogue of a small last layer: tile 16 (up to 64 x
    64), 32 (333 x 513) and 64 (1000 x 777), widths that divide into quads of columns and that do not, batches that leave padded
    columns in the transpose; then a shorter batch on the same buffers.  The gradient is checked against the stored
    activations, and its transpose by what reads it: the bias gradient and the weight gradient."""
    g = torch.Generator().manual_seed(B * 1000 + N)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    K, classes = 24, 7
    seg = api.Segment([K, N], relu, api.MSE_SIL, max_batch=B + 2, dtype=dtype, lr=0.0, momentum=0.0)
    seg.set_params(0, (torch.randn(N, K, generator=g) / math.sqrt(K)).cuda(), torch.randn(N, generator=g).cuda())
    table = torch.rand(classes, N, generator=g).cuda()
    seg.set_labels(table)
    bad = 0
    for rows in (B, max(1, B - 6)):
        X = torch.rand(rows, K, generator=g).to(tdt).cuda()
        if external:
            dA = torch.randn(rows, N, generator=g).to(tdt).cuda()
            seg.step_external(X, dA)
        else:
            y = torch.randint(0, classes, (rows,), generator=g, dtype=torch.int32)
            y[0], y[rows // 2], y[-1] = classes, -3, 1 << 30             # clamped, and their rows counted once each
            bad += len({0, rows // 2, rows - 1})
            loss = float(seg.step(X, y.cuda()))
            assert seg.target_errors() == bad
        A, dZ = seg.get_activation(1, rows), seg.get_activation(1, rows, kind=1)
        live = (A > 0) if relu == api.RELU_ALL else torch.ones_like(A, dtype=torch.bool)
        if external:
            assert torch.equal(dZ, torch.where(live, dA, torch.zeros_like(dA)))
        else:
            diff = A.double() - table.double()[y.clamp(0, classes - 1).long().cuda()]
            mse = float(diff.square().mean())
            assert abs(loss - mse) <= 1e-5 * mse
            ref = torch.where(live, diff * (2.0 / (rows * N)), torch.zeros_like(diff))
            # three float32 roundings, the difference's relative to its terms; bf16 storage: 2^-9 of each element
            err, step = (dZ.double() - ref).abs(), 2.0 ** -22 * 2.0 / (rows * N) * (A.double().abs() + 1.0)
            assert bool((err <= step + (2.0 ** -8 * ref.abs() if dtype == api.BF16 else 0.0)).all())
        # float32 sums of at most 1000 terms: within 1000 2^-24 = 6e-5 of the sum of absolute values, 1e-5 as they are added here
        d = dZ.double()
        assert bool(((seg.get_bias_grad(0).double() - d.sum(0)).abs() <= 1e-5 * d.abs().sum(0) + 1e-30).all())
        dW, bound = d.t() @ X.double(), d.abs().t() @ X.double().abs()
        assert bool(((seg.get_grads(0)[0].double() - dW).abs() <= 1e-5 * bound + 1e-30).all())


@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
@pytest.mark.parametrize("B,w", [(3, 5), (37, 61), (64, 64), (333, 513), (1000, 777), (1001, 776)])
def test_data_gradients_that_nothing_rides_along_with(B, w, dtype):
    """The last layer's in a step from a given gradient (masked, both layouts) and the first layer's of an input gradient (the caller's
    dense matrix), on tiles 16, 32 and 64, against float64 products of the stored factors."""
    g = torch.Generator().manual_seed(B + w)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    N = 50
    X, dA = torch.rand(B, w, generator=g).to(tdt).cuda(), torch.randn(B, N, generator=g).to(tdt).cuda()
    y = torch.randint(0, N, (B,), generator=g, dtype=torch.int32).cuda()
    seg = api.Segment([w, w, N], api.RELU_HIDDEN_IDENTITY_LAST, api.SOFTMAX_XENT, max_batch=B, dtype=dtype, lr=0.0, momentum=0.0, input_grad=True)
    for l, (n, k) in enumerate(((w, w), (N, w))):
        seg.set_params(l, (torch.randn(n, k, generator=g) / math.sqrt(k)).cuda(), torch.randn(n, generator=g).cuda())
    Wop = [seg.get_params(l)[0].to(tdt).double() for l in (0, 1)]

    def check(got, left, right, live):
        # float32 sums of up to 777 terms, 1e-5 of the absolute values as they are added; bf16 storage: 2^-9 of each element
        ref, bound = torch.where(live, left @ right, torch.zeros_like(got, dtype=torch.float64)), left.abs() @ right.abs()
        err = (got.double() - ref).abs()
        assert bool((err <= 1e-5 * bound + (2.0 ** -8 * ref.abs() if dtype == api.BF16 else 0.0)).all())

    seg.step_external(X, dA)
    A1, dZ1 = seg.get_activation(1, B), seg.get_activation(1, B, kind=1)
    check(dZ1, dA.double(), Wop[1], A1 > 0)
    d = dZ1.double()                                  # the transpose, by what reads it
    assert bool(((seg.get_bias_grad(0).double() - d.sum(0)).abs() <= 1e-5 * d.abs().sum(0) + 1e-30).all())
    dX, _ = seg.input_grad(X, y)
    check(dX, seg.get_activation(1, B, kind=1).double(), Wop[0], torch.ones_like(dX, dtype=torch.bool))


@pytest.mark.parametrize("loss", [api.MSE_SIL, api.SOFTMAX_XENT])
@pytest.mark.parametrize("dtype", [api.F32, api.BF16])
def test_replayed_steps_of_more_launches_than_go_one_by_one(dtype, loss):
    """Five small layers come to 10 launches and more, which graphs are still used for: the same bits as eager steps."""
    widths, B, classes = [40, 50, 60, 50, 40, 30], 48, 30
    g = torch.Generator().manual_seed(5)
    tdt = torch.float32 if dtype == api.F32 else torch.bfloat16
    table = torch.rand(classes, widths[-1], generator=g).cuda()
    Xs = [torch.rand(B, widths[0], generator=g).to(tdt).cuda() for _ in range(2)]
    ys = [torch.randint(0, classes, (B,), generator=g, dtype=torch.int32).cuda() for _ in range(2)]
    finals = []
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for graph in (False, True):
            seg = api.Segment(widths, api.RELU_ALL if loss == api.MSE_SIL else api.RELU_HIDDEN_IDENTITY_LAST, loss, max_batch=B, dtype=dtype,
                              lr=0.05, momentum=0.9)
            seg.init(9)
            if loss == api.MSE_SIL:
                seg.set_labels(table)
            seg.set_graph(graph)
            seen = []
            for it in range(7):
                seen.append(seg.step(Xs[it % 2], ys[it % 2]).clone())
                assert seg.graph_stats()[1] == (it if graph else 0)          # all but the first
                if it in (3, 6):                      # reads between replays
                    seen += [t.clone() for l in range(seg.L) for t in seg.get_params(l) + seg.get_momentum(l)]
            stream.synchronize()
            finals.append(seen)
    for a, b in zip(*finals):
        assert torch.equal(a, b)


def test_paced_updates_leave_the_same_bits():
    """A batch above 2048 rows paces the updates of an overlapped step; whoever waits for them ends the pauses."""
    B, widths = 2400, [64, 2304, 2304, 64]
    g = torch.Generator().manual_seed(6)
    table = torch.rand(10, widths[-1], generator=g).cuda()
    X = torch.rand(B, widths[0], generator=g).to(torch.bfloat16).cuda()
    y = torch.randint(0, 10, (B,), generator=g, dtype=torch.int32).cuda()
    finals = []
    for overlap in (False, True):
        seg = api.Segment(widths, api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=api.BF16, lr=0.05, momentum=0.9)
        seg.init(9)
        seg.set_labels(table)
        seg.set_overlap(overlap)
        seen = []
        for it in range(4):
            seen.append(seg.step(X, y).clone())
            if it != 1:
                seen += [t.clone() for l in range(seg.L) for t in seg.get_params(l)]
        finals.append(seen)
    torch.cuda.synchronize()
    for a, b in zip(*finals):
        assert torch.equal(a, b)


@pytest.mark.parametrize("fused", [0, 2])
def test_overlap_leaves_nothing_of_small_layers_pending(fused):
    """The updates of small layers are part of launches in the caller's stream, with overlap on as well: a stream that is being
    captured right behind a step has nothing to wait for, and the graph gives what an eager call gives."""
    B, widths = 64, [96, 128, 64]
    g = torch.Generator().manual_seed(8)
    seg = api.Segment(widths, api.RELU_ALL, api.MSE_SIL, max_batch=B, dtype=api.F32, lr=0.05, momentum=0.9)
    seg.init(9)
    seg.set_labels(torch.rand(10, widths[-1], generator=g).cuda())
    seg.set_fused_update(fused)
    seg.set_overlap(True)
    X = torch.rand(B, widths[0], generator=g).cuda()
    y = torch.randint(0, 10, (B,), generator=g, dtype=torch.int32).cuda()
    out = torch.zeros(B, widths[-1], device="cuda")
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        for _ in range(2):
            seg.step(X, y)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
            seg.forward(X, out=out)
        for _ in range(3):
            out.zero_()
            graph.replay()
            stream.synchronize()
            assert torch.equal(out, seg.forward(X))
            seg.step(X, y)
