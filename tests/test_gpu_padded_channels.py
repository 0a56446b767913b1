"""Layers whose input channels fill no whole 16-byte chunks, which run on a copy
of their input padded to whole ones (or, short ones, on element loads):
channel counts around a piece, a chunk, a K block and several of them, both
forms and types, their input gradients (whole and by phases), the statistics
and the folded epilogue, split and whole launches; against the oracle.  An
infinite pixel stays in its own windows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import assert_close, f64, say

pytestmark = pytest.mark.gpu

DT = {"fp32": torch.float32, "bf16": torch.bfloat16}

# (N, Cin, Cout, H, W, k, stride, pad, dilation)
CASES = ([("bf16", (2, c, 24, 11, 13, 3, 1, 1, 1)) for c in (1, 2, 3, 4, 5, 7, 12, 13, 18, 20, 28, 31, 44)] +
         [("bf16", (1, 66, 72, 9, 8, 3, 1, 1, 1)), ("bf16", (3, 12, 20, 15, 14, 3, 2, 1, 1)),
          ("bf16", (1, 20, 8, 12, 10, 5, 1, 2, 1)), ("bf16", (1, 10, 16, 12, 10, 3, 1, 2, 2)),
          ("bf16", (2, 12, 64, 33, 40, 1, 1, 0, 1)), ("bf16", (2, 60, 64, 20, 20, 1, 1, 0, 1)),
          ("bf16", (1, 7, 8, 12, 11, 3, 2, 1, 2))] +
         [("fp32", (2, c, 12, 11, 13, 3, 1, 1, 1)) for c in (1, 2, 3, 5, 6, 7, 9, 11, 13, 17)] +
         [("fp32", (3, 5, 7, 15, 14, 3, 2, 1, 1)), ("fp32", (1, 33, 18, 9, 8, 3, 1, 1, 1))])


def _inputs(shape, dt, seed):
    N, Cin, Cout, H, W, k, s, p, d = shape
    rng = np.random.default_rng(seed)
    ho, wo = quan.conv_out_size(H, k, s, p, d), quan.conv_out_size(W, k, s, p, d)
    x = torch.from_numpy(rng.standard_normal((N, 4, Cin, H, W), dtype=np.float32)).to(dt)
    w = torch.from_numpy((rng.standard_normal((4, Cout, Cin, k, k)) / np.sqrt(4 * Cin * k * k)).astype(np.float32)).to(dt)
    b = torch.from_numpy((rng.standard_normal((4, Cout)) * 0.3).astype(np.float32)).to(dt)
    dy = torch.from_numpy(rng.standard_normal((N, 4, Cout, ho, wo), dtype=np.float32)).to(dt)
    return x, w, b, dy


@pytest.mark.parametrize("sep", [False, True], ids=["hamilton", "separable"])
@pytest.mark.parametrize("dtype,shape", CASES, ids=[f"{t}-{s}" for t, s in CASES])
def test_padded_channels(dtype, shape, sep):
    say(f"padded channels {dtype} {shape} sep={sep}")
    N, Cin, Cout, H, W, k, s, p, d = shape
    dt = DT[dtype]
    x, w, b, dy = _inputs(shape, dt, sum(shape))
    xg, wg = quan.to_device_layout(x.cuda()), [w[q].contiguous().cuda() for q in range(4)]
    geo = dict(stride=s, pad=p, dilation=d)
    conv = quan.quan_qconv2d_separable_forward if sep else quan.quan_qconv2d_forward
    y = conv(xg, *wg, bias=b.cuda(), **geo)
    # the input gradient contracts over the output channels: swap the roles
    wt = [w[q].transpose(0, 1).contiguous().cuda() for q in range(4)]
    back = quan.quan_qconv2d_separable_backward_data if sep else quan.quan_qconv2d_backward_data
    ho, wo = dy.shape[3:]
    g = torch.from_numpy(np.random.default_rng(7).standard_normal((N, 4, Cin, ho, wo), dtype=np.float32)).to(dt)
    dx = back(quan.to_device_layout(g.cuda()), *wt, (H, W), **geo)
    torch.cuda.synchronize()
    ref = (oracle.qconv2d_separable if sep else oracle.qconv2d)(f64(x), f64(w), f64(b), s, p, d)
    assert_close(f64(y), ref, dt, f"forward {shape}")
    wt64 = np.ascontiguousarray(f64(w).transpose(0, 2, 1, 3, 4))
    ref_fn = oracle.qconv2d_separable_backward if sep else oracle.qconv2d_backward
    ref_dx, _, _ = ref_fn(np.zeros((N, 4, Cout, H, W)), wt64, f64(g), s, p, d)
    assert_close(f64(dx), ref_dx, dt, f"dX {shape}")


# Layers that pad with few channels or in phases (more stages), and 1x1 layers
# on both sides of the rule.
@pytest.mark.parametrize("sep", [False, True], ids=["hamilton", "separable"])
@pytest.mark.parametrize("dtype,shape", [("fp32", (2, c, 12, 13, 11, 5, 1, 2, 1)) for c in (1, 2, 3, 5, 6, 7)] +
                         [("bf16", (2, c, 70, 21, 19, 3, 2, 1, 1)) for c in (69, 100, 133)] +
                         [("bf16", (1, 7, 8, 64, 66, 1, 1, 0, 1)), ("bf16", (1, 15, 130, 70, 80, 1, 1, 0, 1)),
                          ("fp32", (1, 9, 32, 130, 140, 1, 1, 0, 1))], ids=str)
def test_padded_channels_more_stages(dtype, shape, sep):
    test_padded_channels(dtype, shape, sep)


@pytest.mark.parametrize("dtype,cin", [("bf16", 7), ("bf16", 12), ("fp32", 3)])
def test_padded_channels_other_epilogues(dtype, cin):
    say(f"padded channels epilogues {dtype} {cin}")
    dt = DT[dtype]
    shape = (4, cin, 32, 21, 23, 3, 1, 1, 1)
    x, w, b, _ = _inputs(shape, dt, cin)
    rng = np.random.default_rng(3)
    mean, var, gamma, beta = [torch.from_numpy(v.astype(np.float32)) for v in
                              (rng.standard_normal((4, 32)) * 0.5, rng.uniform(0.5, 2.0, (4, 32)),
                               rng.uniform(0.5, 1.5, (4, 32)), rng.standard_normal((4, 32)) * 0.3)]
    xg, wg = quan.to_device_layout(x.cuda()), [w[q].contiguous().cuda() for q in range(4)]
    packed, ws = quan.quan_qconv2d_pack_weights(*wg), tuple(wg[0].shape)
    y = quan.quan_qconv2d_forward_packed(xg, packed, ws, bias=b.cuda(), pad=1)
    z = quan.quan_qconv2d_iqbn_inference(xg, packed, ws, mean.cuda(), var.cuda(), gamma.cuda(), beta.cuda(),
                                         bias=b.cuda(), relu=True, pad=1)
    t, m, v = quan.quan_qconv2d_iqbn_forward(xg, packed, ws, gamma.cuda(), beta.cuda(), bias=b.cuda(), pad=1)
    torch.cuda.synchronize()
    ref = oracle.qconv2d(f64(x), f64(w), f64(b), 1, 1, 1)
    assert_close(f64(z), oracle.iqbn_inference(ref, f64(mean), f64(var), f64(gamma), f64(beta), 1e-5, True), dt, "folded")
    t_ref, m_ref, v_ref = oracle.iqbn(f64(y), f64(gamma), f64(beta), 1e-5, False)
    for got, want, what in ((t, t_ref, "iqbn"), (m, m_ref, "mean"), (v, v_ref, "var")):
        assert_close(f64(got), want, dt, what)


@pytest.mark.parametrize("dtype,cin", [("bf16", 3), ("bf16", 12), ("fp32", 5)])
def test_infinite_pixel_stays_in_its_windows(dtype, cin):
    say(f"padded channels infinity {dtype} {cin}")
    x, w, _, _ = _inputs((1, cin, 8, 9, 10, 3, 1, 1, 1), DT[dtype], 4)
    x[0, :, :, 4, 5] = float("inf")
    y = quan.quan_qconv2d_forward(quan.to_device_layout(x.cuda()), *[w[q].contiguous().cuda() for q in range(4)], pad=1)
    bad = ~torch.isfinite(y[0].float()).all(0).all(0)
    torch.cuda.synchronize()
    want = torch.zeros(9, 10, dtype=torch.bool)
    want[3:6, 4:7] = True
    assert torch.equal(bad.cpu(), want)
