"""Surrogate network kernels on the GPU against the FP64 oracle network.

Element-wise bars.  The library rounds both operands of every product to BF16 and accumulates in
FP32.  Each layer is checked as a function of the GPU's own inputs to it (prefix networks for the
forward pass, single-row gradient calls for the backward pass), against the oracle's layer taking
the same BF16-rounded operands in FP64, with the per-element bound derived in tests/mlp_bounds.py:
FP32 accumulation (gamma_K times the sum of |terms|), tanhf within a few ulp, and BF16 rounding of
an operand only where a rounding midpoint lies within that operand's bound.  Against the unrounded
oracle end to end, the operand rounding itself shows, about sqrt(2) 2^-9 per product compounding
over four layers: that is reported as a relative L2 of at most 3e-2, for context."""
import numpy as np
import pytest

import oracle.mlp as omlp
from tests import mlp_bounds as mb

pytestmark = pytest.mark.gpu

WIDTHS = [5, 256, 256, 256, 64]


bf16 = mb.bf16


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b))


def _data(seed, B, widths=WIDTHS):
    rng = np.random.default_rng(seed)
    X = rng.uniform(-1, 1, size=(B, widths[0])).astype(np.float32)
    t = np.linspace(0, 1, widths[-1])
    Y = (np.sin(np.outer(1 + X[:, 0], 3 * t) + X[:, 1:2]) * (1.5 + X[:, 2:3]) + 0.3 * X[:, 3:4] * X[:, 4:5])
    return X, Y.astype(np.float32)


@pytest.mark.parametrize("M,N,K", [(200, 130, 70), (64, 64, 16), (1, 5, 3), (333, 256, 5)])
def test_gemm_bf16_matches_rounded_product(M, N, K):
    import torch
    from paper_2209_14889_amd import mlp
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((K, N)).astype(np.float32)
    D = mlp.gemm_bf16(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    torch.cuda.synchronize()
    ref = bf16(A) @ bf16(B)
    scale = np.abs(bf16(A)) @ np.abs(bf16(B))
    # FP32 accumulation of K exact BF16 x BF16 products: error <= K 2^-24 sum |a b|
    assert np.all(np.abs(D.cpu().numpy() - ref) <= K * 2.0 ** -24 * scale + 1e-30)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (65, 63, 65), (63, 66, 61), (128, 64, 129), (1, 1, 1), (130, 68, 192)])
def test_gemm_bf16_tile_edges(M, N, K, offset):
    """Sizes at and beside the 64 x 64 x 64 tile, from operands on a 16-byte boundary and 4 bytes past
    one (which takes the scalar loads), against the product of the rounded operands."""
    import torch
    from paper_2209_14889_amd import mlp
    rng = np.random.default_rng(M * 11 + N * 5 + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((K, N)).astype(np.float32)

    def dev(a):
        buf = torch.empty(a.size + offset, dtype=torch.float32, device="cuda")
        v = buf[offset:].view(*a.shape)
        v.copy_(torch.from_numpy(a))
        return v

    D = mlp.gemm_bf16(dev(A), dev(B))
    torch.cuda.synchronize()
    scale = np.abs(bf16(A)) @ np.abs(bf16(B))
    # FP32 accumulation of K exact BF16 x BF16 products: error <= K 2^-24 sum |a b|
    assert np.all(np.abs(D.cpu().numpy() - bf16(A) @ bf16(B)) <= K * 2.0 ** -24 * scale + 1e-30)


@pytest.mark.parametrize("M,N,K", [(2, 20_000_004, 65), (3, 9_000_001, 66), (66, 1, 9_000_001), (65, 2, 20_000_004)])
def test_gemm_bf16_rows_beyond_a_tiles_buffer_range(M, N, K):
    """Rows so long that 64 of them pass 2^31 and 2^32 bytes, of either operand, from 16-byte and scalar
    loads.  Small whole numbers: every product and sum is exact, so the result is too."""
    import torch
    from paper_2209_14889_amd import mlp
    rng = np.random.default_rng(M + N + K)

    def whole(*shape):
        return torch.from_numpy(rng.integers(-3, 4, shape).astype(np.float32)).cuda()

    if N > K:
        row = torch.arange(N, device="cuda", dtype=torch.int32) % 7 - 3
        A, B = whole(M, K), torch.empty((K, N), dtype=torch.float32, device="cuda")
        for k in range(K):
            B[k] = torch.roll(row, k)
        want = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        for m in range(M):
            for k in range(K):
                want[m] += A[m, k] * B[k]
    else:
        at = torch.from_numpy(np.unique(np.r_[0, 1, K // 2, K - 2, K - 1, rng.integers(0, K, 50)])).cuda()
        A, B = torch.zeros((M, K), dtype=torch.float32, device="cuda"), whole(K, N)
        A[:, at] = whole(M, at.numel()).abs() + 1
        want = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        for j in at.tolist():
            want += A[:, j:j + 1] * B[j:j + 1]
    assert torch.equal(mlp.gemm_bf16(A, B), want)


@pytest.mark.parametrize("K", [1, 4, 5, 8, 15, 16, 17])
@pytest.mark.parametrize("batch,offset", [(1, 0), (64, 0), (65, 1), (130, 0)])
def test_layer_of_few_inputs(K, batch, offset):
    """One layer of up to and just beyond 16 inputs, too wide for the one-launch form, from inputs on a 16-byte
    boundary and 4 bytes past one, element by element against the layer of the rounded operands."""
    import torch
    from paper_2209_14889_amd import mlp
    N = 516
    rng = np.random.default_rng(100 * K + batch)
    X = rng.uniform(-1, 1, (batch, K)).astype(np.float32)
    W, b = rng.uniform(-1, 1, (N, K)).astype(np.float32), rng.uniform(-1, 1, N).astype(np.float32)
    buf = torch.empty(X.size + offset, dtype=torch.float32, device="cuda")
    x = buf[offset:].view(batch, K)
    x.copy_(torch.from_numpy(X))
    net = mlp.MLP([K, N], batch)
    net.set_params(np.concatenate([W.ravel(), b]))
    Y = net.forward(x).cpu().numpy().astype(np.float64)
    z, ez = mb.layer_bound(X.astype(np.float64), np.zeros(X.shape), W.astype(np.float64), b.astype(np.float64))
    assert np.all(np.abs(Y - z) <= ez)
    net.close()


@pytest.mark.parametrize("widths,batch", [
    ([5, 256, 256, 256, 64], 1), ([5, 256, 256, 256, 64], 17), ([5, 256, 256, 256, 64], 4097),
    ([5, 256, 256, 256, 64], 8193 + 15), ([3, 512, 20, 512, 1], 33), ([130, 4], 5), ([7, 300, 100, 65], 70),
    ([5, 384, 384, 16], 8200), ([5, 100, 513, 16], 40), ([5, 30, 40, 16], 40)])
def test_one_launch_forward_is_the_layers_forward(widths, batch):
    """The forward pass of narrow networks in one launch (both entry points, all three row counts per
    block, ragged tiles and panels) against the same layers one launch each, which a call whose output
    overlaps its input takes: the same bits.  The last two networks (a layer too wide, rows not on 16
    bytes) take the layers in every call."""
    import torch
    from paper_2209_14889_amd import lb, mlp
    params = mlp.init_params(widths, 31)
    rng, o = np.random.default_rng(batch), 0
    for a, b in zip(widths[:-1], widths[1:]):
        o += a * b
        params[o:o + b] = rng.uniform(-0.1, 0.1, b)
        o += b
    X = torch.from_numpy(rng.uniform(-1, 1, (batch, widths[0])).astype(np.float32)).cuda()
    net = mlp.MLP(widths, batch)
    net.set_params(params)
    Y = net.forward(X).cpu().numpy()
    if batch * max(widths[1:-1], default=0) <= 1 << 19:
        Yn = torch.empty((batch, widths[-1]), dtype=torch.float32, device="cuda")
        mlp.forward_noalloc(widths, torch.from_numpy(params).cuda(), X, Yn)
        torch.cuda.synchronize()
        assert np.array_equal(Yn.cpu().numpy(), Y)
    both = torch.empty(batch * max(widths[0], widths[-1]), dtype=torch.float32, device="cuda")
    both[:X.numel()] = X.flatten()
    torch.cuda.synchronize()
    lb.check(mlp.lib().lb_mlp_forward(net.h, mlp._dev(both), batch, mlp._dev(both)))
    net.stream.synchronize()
    assert np.array_equal(both[:Y.size].cpu().numpy().reshape(Y.shape), Y)
    net.close()


def _net(params, B=512):
    from paper_2209_14889_amd import mlp
    net = mlp.MLP(WIDTHS, B)
    net.set_params(params)
    return net


def _prefix_preactivations(params, X):
    """The GPU's pre-activation of every layer for the rows X: the network of the first k layers
    returns the full network's k-th pre-activation bit for bit (same kernels, same data)."""
    import torch
    from paper_2209_14889_amd import mlp
    zs = []
    for k in range(1, len(WIDTHS)):
        net = mlp.MLP(WIDTHS[:k + 1], X.shape[0])
        net.set_params(mb.prefix_params(params, WIDTHS, k))
        zs.append(net.forward(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64))
        net.close()
    return zs


def _gpu_layer_inputs(params, X, zs):
    """Reference of every layer on the GPU's inputs, checked element by element; returns the layer
    inputs (FP64 tanh of the GPU's pre-activations) and their bounds."""
    layers = omlp.unpack(np.asarray(params, np.float64), WIDTHS)
    A, EA = X.astype(np.float64), np.zeros(X.shape)
    acts, errs = [A], [EA]
    for l, (W, b) in enumerate(layers):
        z, ez = mb.layer_bound(A, EA, W, b)
        bad = np.abs(zs[l] - z) > ez
        print(f"  layer {l}: max |gpu - ref| / bound {np.max(np.abs(zs[l] - z) / ez):.3f}, "
              f"median bound / max |z| {np.median(ez) / np.max(np.abs(z)):.1e}", flush=True)
        assert not bad.any(), (l, int(bad.sum()))
        if l + 1 < len(layers):
            A, EA = mb.hidden(zs[l])
            acts.append(A)
            errs.append(EA)
    return acts, errs


def test_forward_matches_oracle():
    import torch
    from paper_2209_14889_amd import mlp
    params = mlp.init_params(WIDTHS, 11)
    rng, o = np.random.default_rng(4), 0
    for l in range(4):          # non-zero biases
        o += WIDTHS[l + 1] * WIDTHS[l]
        params[o:o + WIDTHS[l + 1]] = rng.uniform(-0.1, 0.1, WIDTHS[l + 1])
        o += WIDTHS[l + 1]
    X, _ = _data(5, 300)
    net = _net(params)
    Y = net.forward(torch.from_numpy(X).cuda()).cpu().numpy()
    assert Y.shape == (300, 64)
    assert np.array_equal(net.get_params(), params)
    net.close()
    zs = _prefix_preactivations(params, X)
    assert np.array_equal(zs[-1], Y.astype(np.float64))   # the full network is its own last prefix
    _gpu_layer_inputs(params, X, zs)                         # every layer, every element
    assert rel(Y, omlp.forward(params, WIDTHS, X, mb.bf16)[-1]) < 2e-3
    assert rel(Y, omlp.forward(params, WIDTHS, X)[-1]) < 3e-2


def _unpack_grads(flat):
    return omlp.unpack(np.asarray(flat, np.float64), WIDTHS)


def test_gradients_match_oracle():
    """Gradients of a 256-row batch.  Each row alone (batch 1) exposes its pre-activation gradients
    as the bias gradients, so every backward layer is checked element by element on the GPU's own
    inputs; the batch of 2^8 rows then holds exactly those values times 2^-8, and its weight and
    bias gradients are checked element by element as sums over the rows."""
    import torch
    from paper_2209_14889_amd import mlp
    params = mlp.init_params(WIDTHS, 12)
    B = 256
    X, Y = _data(6, B)
    zs = _prefix_preactivations(params, X)
    acts, errs = _gpu_layer_inputs(params, X, zs)
    layers = omlp.unpack(np.asarray(params, np.float64), WIDTHS)
    L = len(layers)
    net = _net(params, B)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    # one row at a time
    dz_rows = [[None] * B for _ in range(L)]
    worst = 0.0
    for r in range(B):
        _, g1 = net.gradients(Xd[r:r + 1], Yd[r:r + 1])
        g1 = _unpack_grads(g1)
        for l in range(L):
            dz_rows[l][r] = g1[l][1][None, :]
        dz, edz = mb.output_grad_bound(zs[-1][r:r + 1], Y[r:r + 1], 1)
        assert np.all(np.abs(dz_rows[L - 1][r] - dz) <= edz), r
        for l in range(L - 1, -1, -1):
            A, EA = acts[l][r:r + 1], errs[l][r:r + 1]
            gW, egW, gb, egb, dzp, edzp = mb.backward_layer_bound(dz_rows[l][r], A, EA, layers[l][0], l == 0)
            assert np.all(np.abs(g1[l][0] - gW) <= egW), (r, l)
            worst = max(worst, float(np.max(np.abs(g1[l][0] - gW) / np.maximum(egW, 1e-300))))
            if l > 0:
                assert np.all(np.abs(dz_rows[l - 1][r] - dzp) <= edzp), (r, l)
    print(f"  single rows: max |gpu - ref| / bound {worst:.3f}", flush=True)
    # the whole batch: each row's values scaled by exactly 2^-8
    loss, g = net.gradients(Xd, Yd)
    g = _unpack_grads(g)
    for l in range(L):
        dz = np.concatenate(dz_rows[l]) / B
        gW, egW, gb, egb, _, _ = mb.backward_layer_bound(dz, acts[l], errs[l], layers[l][0], True)
        assert np.all(np.abs(g[l][0] - gW) <= egW), l
        assert np.all(np.abs(g[l][1] - gb) <= egb), l
        print(f"  batch layer {l}: max |gpu - ref| / bound {np.max(np.abs(g[l][0] - gW) / egW):.3f}, "
              f"median bound / max |dW| {np.median(egW) / np.max(np.abs(gW)):.1e}", flush=True)
    # end to end against the oracle network (context: the rounding of every operand to BF16)
    g_flat = np.concatenate([np.concatenate([gW.ravel(), gb]) for gW, gb in g])
    assert rel(g_flat, omlp.gradients(params, WIDTHS, X, Y, mb.bf16)) < 2e-3
    assert rel(g_flat, omlp.gradients(params, WIDTHS, X, Y)) < 3e-2
    assert abs(loss - omlp.loss(params, WIDTHS, X, Y)) < 3e-2 * omlp.loss(params, WIDTHS, X, Y)
    # deterministic: the same call gives the same bits
    loss2, g2 = net.gradients(Xd, Yd)
    assert loss2 == loss and np.array_equal(_unpack_grads(g2)[0][0], g[0][0])
    net.close()


@pytest.mark.parametrize("widths,batch", [
    ([5, 256, 256, 256, 64], 256), ([5, 256, 256, 256, 64], 1), ([5, 64, 64, 64, 16], 65), ([7, 300, 100, 65], 70),
    ([3, 512, 20, 512, 1], 33), ([130, 36], 17), ([5, 30, 30, 30, 16], 40), ([16, 520, 520, 520, 33], 100)])
def test_gradients_in_three_launches_and_layer_by_layer(widths, batch):
    """Gradients and one training step with an arena that holds a gradient buffer per layer (narrow
    networks: three launches; the last two networks: a launch per layer, then all weight gradients)
    against an arena of the least accepted size (two gradient buffers, a launch per layer): the same
    products in the same order, so the same gradients bit for bit; and against the oracle network with
    the same operand rounding.  The update differs at most by the rounding of about ten operations on
    a step of size lr, and of the new parameter."""
    import ctypes

    import torch
    from paper_2209_14889_amd import lb, mlp
    params = mlp.init_params(widths, 41)
    rng = np.random.default_rng(42)
    X = rng.uniform(-1, 1, (batch, widths[0])).astype(np.float32)
    Y = rng.uniform(0.5, 1.5, (batch, widths[-1])).astype(np.float32)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    full = mlp.MLP(widths, batch)
    wmax = max(widths)
    hidden = sum(widths[1:-1])
    less = 4 * max(0, hidden - 2 * wmax) * batch // 256 * 256
    small = mlp.MLP(widths, batch)
    lb.check(mlp.lib().lb_mlp_destroy(small.h))
    h = ctypes.c_void_p()
    lb.check(mlp.lib().lb_mlp_create(ctypes.byref(small.cfg), mlp._dev(small.arena),
                                     ctypes.c_size_t(small.arena.numel() - less),
                                     ctypes.c_void_p(small.stream.cuda_stream), ctypes.byref(h)))
    small.h = h
    out = []
    lr = 1e-3
    for net in (full, small):
        net.set_params(params)
        loss, g = net.gradients(Xd, Yd)
        net.train_step(Xd, Yd, lr)
        out.append((loss, g, net.get_params()))
        net.close()
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1])
    u = 2.0 ** -24
    assert np.all(np.abs(out[0][2].astype(np.float64) - out[1][2]) <= 16 * u * lr + u * np.abs(out[1][2]))
    assert rel(out[0][1], omlp.gradients(params, widths, X, Y, mb.bf16)) < 2e-3
    Yh = omlp.forward(params, widths, X, mb.bf16)[-1]
    loss = np.mean(np.sum((Yh - Y) ** 2, axis=1) / np.sum(Y.astype(np.float64) ** 2, axis=1))
    assert abs(out[0][0] - loss) < 2e-3 * loss


@pytest.mark.parametrize("widths,batch", [
    ([5, 16, 16, 8], 16385), ([3, 8, 8, 2], 16400), ([5, 64, 64, 8], 32769), ([4, 100, 8], 32800), ([6, 40], 300)])
def test_forward_of_many_rows_is_the_forward_of_few(widths, batch):
    """Just beyond the rows that thin networks take in one launch (and, for the last two, with no such limit,
    and with one layer): the same bits as the same rows a thousand at a time."""
    import torch
    from paper_2209_14889_amd import mlp
    rng = np.random.default_rng(batch)
    X = torch.from_numpy(rng.uniform(-1, 1, (batch, widths[0])).astype(np.float32)).cuda()
    net = mlp.MLP(widths, batch)
    net.set_params(mlp.init_params(widths, 33))
    Y = net.forward(X)
    parts = torch.cat([net.forward(X[i:i + 1000]) for i in range(0, batch, 1000)])
    assert torch.equal(Y, parts)
    net.close()


@pytest.mark.parametrize("widths,batch", [([5, 64, 64, 64, 8], 8192), ([5, 64, 64, 64, 8], 8193), ([5, 384, 384, 384, 8], 4096),
                                          ([5, 384, 384, 384, 8], 4097), ([200, 200, 200, 200, 8], 300), ([6, 40], 70)])
def test_gradients_on_either_side_of_the_one_launch_form(widths, batch):
    """The most rows that gradients take in three launches, one more, and networks that never do."""
    test_gradients_in_three_launches_and_layer_by_layer(widths, batch)


def test_first_adam_step_follows_its_definition():
    import torch
    from paper_2209_14889_amd import mlp
    params = mlp.init_params(WIDTHS, 13)
    X, Y = _data(7, 128)
    net = _net(params)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    _, g = net.gradients(Xd, Yd)
    lr = 1e-3
    net.train_step(Xd, Yd, lr)
    p1 = net.get_params()
    # step 1 with bias correction: m_hat = g, v_hat = g^2
    g64 = g.astype(np.float64)
    expect = params - lr * g64 / (np.abs(g64) + 1e-8)
    assert np.max(np.abs(p1 - expect)) < 1e-6
    net.close()


def test_training_reduces_the_loss():
    import torch
    from paper_2209_14889_amd import mlp
    X, Y = _data(8, 1024)
    net = _net(mlp.init_params(WIDTHS, 14), 256)
    Xd, Yd = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    l0, _ = net.gradients(Xd[:256], Yd[:256])
    for it in range(400):
        b = (it % 4) * 256
        net.train_step(Xd[b:b + 256], Yd[b:b + 256], 1e-3)
    net.stream.synchronize()
    l1, _ = net.gradients(Xd[:256], Yd[:256])
    assert l1 < 0.05 * l0, (l0, l1)
    net.close()


def test_rejects_oversized_batch():
    import torch
    from paper_2209_14889_amd import lb
    net = _net(np.zeros(sum(WIDTHS[i] * WIDTHS[i + 1] + WIDTHS[i + 1] for i in range(4)), np.float32), 64)
    with pytest.raises(lb.LBError):
        net.forward(torch.zeros((65, 5), device="cuda"))
    net.close()


def test_surrogate_pipeline_small():
    """End to end at reduced size (64^2 lattices, 1024 steps, 16 samples): LB data from batched
    ensembles, an ensemble of networks trained by the library, and the fallback rule: rows over the
    threshold are the LB's own values, bit for bit."""
    from paper_2209_14889_amd import surrogate as sg
    kw = dict(n=64, steps=1024, every=64)
    train = list(range(3000, 3096))
    test = list(range(9000, 9016))
    inp, Y = sg.simulate(train, batch=48, **kw)
    assert Y.shape == (96, 16) and np.all(np.isfinite(Y))
    assert np.abs(Y).max() > 0
    s = sg.Surrogate(members=2, widths=[5, 64, 64, 16], max_batch=96)
    s.fit(sg.features(inp), Y, epochs=40, batch=32)
    th = s.calibrate(sg.features(inp[:48]), Y[:48])
    assert th >= 0.0
    s.threshold = float(np.median(s.predict(sg.features([sg.wl.surrogate_inputs(x) for x in test]))[1]))
    out, info = s.predict_with_fallback(test, batch=16, **kw)
    fb = info["fallback"]
    assert 0 < fb.size < len(test)
    _, Yt = sg.simulate(test, batch=16, **kw)
    assert np.array_equal(out[fb], Yt[fb])


def test_surrogate_gains_over_lb():
    """What the trained network buys, at reduced training size (512 LB runs of the full 128^2,
    4096-step protocol; 64 held-out runs): its restoring-force series are within a few per cent
    of the LB's (median <= 2%, 90th percentile <= 4%), and predicting them costs a small
    fraction of simulating them."""
    import time

    import torch
    from paper_2209_14889_amd import surrogate as sg
    inp, Y = sg.simulate(range(3000, 3512), batch=512)
    s = sg.Surrogate(members=2, max_batch=128)
    s.fit(sg.features(inp), Y, epochs=800, batch=128)
    test = list(range(9000, 9064))
    Xt = sg.features([sg.wl.surrogate_inputs(x) for x in test])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _, Yt = sg.simulate(test, batch=64)
    t_lb = time.perf_counter() - t0
    s.predict(Xt)
    t0 = time.perf_counter()
    mean, _ = s.predict(Xt)
    t_inf = time.perf_counter() - t0
    err = np.linalg.norm(mean - Yt, axis=1) / np.linalg.norm(Yt, axis=1)
    print(f"median error {np.median(err):.4f}, p90 {np.quantile(err, 0.9):.4f}, LB {t_lb:.3f} s, "
          f"network {t_inf * 1e3:.2f} ms", flush=True)
    assert np.median(err) <= 0.02 and np.quantile(err, 0.9) <= 0.04
    assert t_lb > 20 * t_inf
