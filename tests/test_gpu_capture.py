"""Graphs captured on a stream that has run the layer with another batch:
replays, with eager work between them, equal the eager result."""
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import assert_close, f64, say

pytestmark = pytest.mark.gpu


def _maps(seed, *shape):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(*shape, generator=g)


def _capture(stream, fn):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        fn()
    return graph


@pytest.mark.parametrize("dtype,c,o,k,warm,n", [("bf16", 32, 48, 3, 1, 6), ("bf16", 32, 48, 3, 6, 1),
                                                ("fp32", 8, 24, 3, 1, 4), ("bf16", 64, 64, 1, 1, 5)])
def test_inference_of_another_batch(dtype, c, o, k, warm, n):
    say(f"capture of an inference layer {dtype} {c}->{o} k{k} batch {warm} then {n}")
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    x = _maps(1, max(n, warm), 4, c, 28, 27).to(dt)
    w = (_maps(2, 4, o, c, k, k) * 0.1).to(dt)
    mean, gamma, beta = _maps(3, 3, 4, o)
    var = _maps(4, 4, o).abs() + 0.5
    packed = quan.quan_qconv2d_pack_weights(*[w[q].contiguous().cuda() for q in range(4)])
    params = [t.contiguous().cuda() for t in (mean, var, gamma, beta)]
    small, xg = [quan.to_device_layout(x[:m].cuda()) for m in (warm, n)]
    out = quan.empty_qmap(n, o, 28, 27, dt, xg.device)

    def run(t, **kw):
        return quan.quan_qconv2d_iqbn_inference(t, packed, tuple(w.shape[1:]), *params, pad=k // 2, relu=True, **kw)

    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        run(small)
    torch.cuda.synchronize()
    graph = _capture(st, lambda: run(xg, out=out))
    ref = oracle.iqbn_inference(oracle.qconv2d(f64(x[:n]), f64(w), None, 1, k // 2, 1), f64(mean), f64(var), f64(gamma),
                                f64(beta), 1e-5, True)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert_close(f64(out), ref, dt, "replay")
        with torch.cuda.stream(st):
            eager = run(xg)
        torch.cuda.synchronize()
        assert_close(f64(eager), ref, dt, "eager")


def test_weight_gradient_captured_then_outgrown():
    """The partial sums' buffer of a captured weight gradient outlives a larger
    layer's call on the stream."""
    say("capture of a weight gradient, then a larger call")
    bf = torch.bfloat16
    x, dy = [quan.to_device_layout(_maps(i, 4, 4, 16, 20, 21).to(bf).cuda()) for i in (1, 2)]
    bx, bdy = [quan.to_device_layout(_maps(i, 4, 4, 128, 30, 30).to(bf).cuda()) for i in (3, 4)]
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        want, wb = quan.quan_qconv2d_backward_weight(x, dy, (3, 3), pad=1)
    torch.cuda.synchronize()
    held = []
    graph = _capture(st, lambda: held.append(quan.quan_qconv2d_backward_weight(x, dy, (3, 3), pad=1)))
    with torch.cuda.stream(st):
        big, _ = quan.quan_qconv2d_backward_weight(bx, bdy, (3, 3), pad=1)
    torch.cuda.synchronize()
    filler = [torch.full((1 << 20,), float("nan"), device="cuda") for _ in range(16)]
    for _ in range(3):
        dw, db = held[0]
        for t in (*dw, db):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((*dw, db), (*want, wb)))
        with torch.cuda.stream(st):
            again, _ = quan.quan_qconv2d_backward_weight(bx, bdy, (3, 3), pad=1)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(again, big))
    assert all(bool(t.isnan().all()) for t in filler)


def test_training_layer_of_a_smaller_batch():
    """Warmed up with statistics in the epilogue, captured with the separate
    pass of a few pixels."""
    say("capture of a training layer, batch 8 then 1")
    bf = torch.bfloat16
    x = _maps(1, 8, 4, 48, 32, 32).to(bf)
    w = (_maps(2, 4, 32, 48, 3, 3) * 0.05).to(bf)
    gamma, beta = (_maps(3, 2, 4, 32).sigmoid() + 0.5).cuda()
    packed = quan.quan_qconv2d_pack_weights(*[w[q].contiguous().cuda() for q in range(4)])
    big, xg = [quan.to_device_layout(x[:m].cuda()) for m in (8, 1)]
    out = quan.empty_qmap(1, 32, 16, 16, bf, xg.device)
    mean, var = torch.empty(2, 4, 32, device="cuda")

    def run(t, **kw):
        return quan.quan_qconv2d_iqbn_forward(t, packed, (32, 48, 3, 3), gamma, beta, stride=2, pad=1, **kw)

    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        run(big)
    torch.cuda.synchronize()
    graph = _capture(st, lambda: run(xg, out=out, mean=mean, var=var))
    # the captured layer sums K in one piece, an eager one of this size in
    # several: equal up to the rounding of the convolution's output to bf16
    # (half an ulp, 2^-9 of |y| <= 4.5 sigma, times gamma / sigma <= 1.5: 0.4 of
    # the bar at |z| = 6, the mean of y being near 0) and of z itself
    refs = oracle.iqbn(oracle.qconv2d(f64(x[:1]), f64(w), None, 2, 1, 1), f64(gamma), f64(beta), 1e-5, False)
    for _ in range(3):
        for t in (out, mean, var):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for t, ref, what in zip((out, mean, var), refs, ("out", "mean", "var")):
            assert_close(f64(t), ref, bf, f"{what} of the replay")
        with torch.cuda.stream(st):
            run(big)
        torch.cuda.synchronize()


def test_weight_gradient_of_a_smaller_batch():
    """More slices for 3 images than for 4: the stream that has run 4 is
    captured with 3."""
    say("capture of a weight gradient, batch 4 then 3")
    bf = torch.bfloat16
    x, dy = [quan.to_device_layout(_maps(i, 4, 4, c, 32, 32).to(bf).cuda()) for i, c in ((1, 32), (2, 8))]
    xs, dys = x[:3], dy[:3]
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    want, wb = quan.quan_qconv2d_backward_weight(xs, dys, (3, 3), pad=1)
    with torch.cuda.stream(st):
        quan.quan_qconv2d_backward_weight(x, dy, (3, 3), pad=1)
    torch.cuda.synchronize()
    held = []
    graph = _capture(st, lambda: held.append(quan.quan_qconv2d_backward_weight(xs, dys, (3, 3), pad=1)))
    for _ in range(3):
        dw, db = held[0]
        for t in (*dw, db):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((*dw, db), (*want, wb)))
        with torch.cuda.stream(st):
            quan.quan_qconv2d_backward_weight(x, dy, (3, 3), pad=1)
        torch.cuda.synchronize()
