"""Convolutions of few output pixels, whose K loop is split over work-groups
(fp32 partial tiles, added by a second launch that applies the epilogue):
both types, whole and partial channel chunks, output channels that are no
multiple of four, pixel counts around a tile, several channel tiles, stage
counts that do not divide, with the bias, the folded inference map, IQBN
behind it, and as input gradients with and without phases; against the
oracle.  Under graph capture without a warm-up on that size the layer runs
unsplit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import assert_close, f64, say

pytestmark = pytest.mark.gpu

DT = {"fp32": torch.float32, "bf16": torch.bfloat16}

# (N, Cin, Cout, H, W, k, stride, pad, dilation)
SHAPES = [
    (1, 64, 64, 1, 1, 3, 1, 1, 1),       # one pixel
    (1, 128, 32, 5, 6, 3, 1, 1, 1),
    (1, 128, 40, 4, 32, 3, 1, 1, 1),     # 128 pixels
    (1, 72, 100, 3, 43, 3, 1, 1, 1),     # 129; two or more channel tiles; odd block count
    (2, 100, 30, 9, 7, 3, 1, 1, 1),      # partial chunks, c_out % 4 != 0
    (1, 67, 13, 7, 7, 3, 1, 1, 1),
    (1, 256, 256, 7, 7, 3, 2, 1, 1),
    (1, 512, 24, 6, 6, 1, 1, 0, 1),      # 1x1
    (1, 96, 64, 9, 9, 3, 1, 2, 2),       # dilation
    (1, 64, 24, 9, 9, 5, 1, 2, 1),
]


def _inputs(shape, dt, seed):
    N, Cin, Cout, H, W, k, s, p, d = shape
    rng = np.random.default_rng(seed)
    x = torch.from_numpy(rng.standard_normal((N, 4, Cin, H, W), dtype=np.float32)).to(dt)
    w = torch.from_numpy((rng.standard_normal((4, Cout, Cin, k, k)) / np.sqrt(4 * Cin * k * k)).astype(np.float32)).to(dt)
    b = torch.from_numpy((rng.standard_normal((4, Cout)) * 0.3).astype(np.float32)).to(dt)
    f = [torch.from_numpy(v.astype(np.float32)) for v in
         (rng.standard_normal((4, Cout)) * 0.5, rng.uniform(0.5, 2.0, (4, Cout)), rng.uniform(0.5, 1.5, (4, Cout)),
          rng.standard_normal((4, Cout)) * 0.3)]
    return x, w, b, f


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_split_forward(shape, dtype):
    say(f"split convolution {dtype} {shape}")
    N, Cin, Cout, H, W, k, s, p, d = shape
    dt = DT[dtype]
    x, w, b, (mean, var, gamma, beta) = _inputs(shape, dt, sum(shape))
    xg, wg = quan.to_device_layout(x.cuda()), [w[q].contiguous().cuda() for q in range(4)]
    geo = dict(stride=s, pad=p, dilation=d)
    packed = quan.quan_qconv2d_pack_weights(*wg)
    y = quan.quan_qconv2d_forward(xg, *wg, bias=b.cuda(), **geo)
    plain = quan.quan_qconv2d_forward_packed(xg, packed, tuple(wg[0].shape), **geo)
    z = quan.quan_qconv2d_iqbn_inference(xg, packed, tuple(wg[0].shape), mean.cuda(), var.cuda(), gamma.cuda(),
                                         beta.cuda(), bias=b.cuda(), relu=True, **geo)
    t, m, v = quan.quan_qconv2d_iqbn_forward(xg, packed, tuple(wg[0].shape), gamma.cuda(), beta.cuda(), bias=b.cuda(),
                                             **geo)
    torch.cuda.synchronize()
    ref = oracle.qconv2d(f64(x), f64(w), f64(b), s, p, d)
    assert_close(f64(y), ref, dt, f"bias {shape}")
    assert_close(f64(plain), oracle.qconv2d(f64(x), f64(w), None, s, p, d), dt, f"plain {shape}")
    assert_close(f64(z), oracle.iqbn_inference(ref, f64(mean), f64(var), f64(gamma), f64(beta), 1e-5, True), dt,
                 f"folded {shape}")
    t_ref, m_ref, v_ref = oracle.iqbn(f64(y), f64(gamma), f64(beta), 1e-5, False)
    assert_close(f64(m), m_ref, dt, f"mean {shape}")
    assert_close(f64(v), v_ref, dt, f"var {shape}")
    if y.shape[0] * y.shape[3] * y.shape[4] > 4:
        assert_close(f64(t), t_ref, dt, f"iqbn {shape}")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_split_input_gradient(shape, dtype):
    say(f"split input gradient {dtype} {shape}")
    N, Cin, Cout, H, W, k, s, p, d = shape
    Cin, Cout = Cout, Cin  # the contraction runs over the output channels
    dt = DT[dtype]
    rng = np.random.default_rng(sum(shape))
    ho, wo = quan.conv_out_size(H, k, s, p, d), quan.conv_out_size(W, k, s, p, d)
    w = torch.from_numpy((rng.standard_normal((4, Cout, Cin, k, k)) / np.sqrt(4 * Cout * k * k)).astype(np.float32)).to(dt)
    dy = torch.from_numpy(rng.standard_normal((N, 4, Cout, ho, wo), dtype=np.float32)).to(dt)
    dx = quan.quan_qconv2d_backward_data(quan.to_device_layout(dy.cuda()), *[w[q].contiguous().cuda() for q in range(4)],
                                         (H, W), stride=s, pad=p, dilation=d)
    torch.cuda.synchronize()
    ref, _, _ = oracle.qconv2d_backward(np.zeros((N, 4, Cin, H, W)), f64(w), f64(dy), s, p, d)
    assert_close(f64(dx), ref, dt, f"dX {shape}")


def test_split_under_capture_without_warm_up():
    """The partial tiles need memory that a capturing stream cannot get: the
    layer then runs unsplit, inside the capture; replays equal eager runs up
    to the order of the sums."""
    say("split convolution under capture")
    shape = (1, 192, 96, 6, 7, 3, 1, 1, 1)
    x, w, _, _ = _inputs(shape, torch.bfloat16, 9)
    packed = quan.quan_qconv2d_pack_weights(*[w[q].contiguous().cuda() for q in range(4)])
    wshape = tuple(w.shape[1:])
    xg = quan.to_device_layout(x.cuda())
    out = quan.empty_qmap(1, 96, 6, 7, torch.bfloat16, torch.device("cuda:0"))
    st = torch.cuda.Stream()
    # one unsplit size on this stream first: the library's other buffers
    big = quan.to_device_layout(torch.randn(64, 4, 32, 32, 32).to(torch.bfloat16).cuda())
    wb = [torch.randn(64, 32, 3, 3).to(torch.bfloat16).cuda() for _ in range(4)]
    pb = quan.quan_qconv2d_pack_weights(*wb)
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        quan.quan_qconv2d_forward_packed(big, pb, (64, 32, 3, 3), pad=1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        quan.quan_qconv2d_forward_packed(xg, packed, wshape, pad=1, out=out)
    ref = oracle.qconv2d(f64(x), f64(w), None, 1, 1, 1)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert_close(f64(out), ref, torch.bfloat16, "replay")
        eager = quan.quan_qconv2d_forward_packed(xg, packed, wshape, pad=1)
        torch.cuda.synchronize()
        assert_close(f64(eager), ref, torch.bfloat16, "eager")


def test_captured_buffer_outlives_a_larger_call():
    """A graph captured after a warm-up holds the partial tiles' buffer; a
    later, larger layer on the same stream takes a new one and the replays go
    on giving the same result."""
    say("split convolution captured, then outgrown")
    x, w, _, _ = _inputs((1, 192, 96, 6, 7, 3, 1, 1, 1), torch.bfloat16, 9)
    packed = quan.quan_qconv2d_pack_weights(*[w[q].contiguous().cuda() for q in range(4)])
    xg, wshape = quan.to_device_layout(x.cuda()), tuple(w.shape[1:])
    out = quan.empty_qmap(1, 96, 6, 7, torch.bfloat16, torch.device("cuda:0"))
    big, wb, _, _ = _inputs((1, 256, 256, 20, 20, 3, 1, 1, 1), torch.bfloat16, 10)
    bigg, pb = quan.to_device_layout(big.cuda()), quan.quan_qconv2d_pack_weights(*[wb[q].contiguous().cuda() for q in range(4)])
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        eager = quan.quan_qconv2d_forward_packed(xg, packed, wshape, pad=1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        quan.quan_qconv2d_forward_packed(xg, packed, wshape, pad=1, out=out)
    with torch.cuda.stream(st):
        y = quan.quan_qconv2d_forward_packed(bigg, pb, tuple(wb.shape[1:]), pad=1)
    torch.cuda.synchronize()
    filler = [torch.full((1 << 20,), float("nan"), device="cuda") for _ in range(8)]
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        with torch.cuda.stream(st):
            again = quan.quan_qconv2d_forward_packed(bigg, pb, tuple(wb.shape[1:]), pad=1)
        torch.cuda.synchronize()
        assert torch.equal(again, y)
    assert all(bool(t.isnan().all()) for t in filler)
