"""Weight gradients of the layers that the row kernel takes (at most 16
channels; bf16 channel counts that are no multiple of 8; fp32 ones that save
half the padded work) and of the four-component kernel's 32-channel tiles,
against the oracle's fp64 gradients, at the edges of its plan: output widths
around a quad of pixels, a segment and a chunk, tap groups of one to three,
strides and dilations with and without a shared window, one and several
tiles, odd channel counts (8-byte pieces).

Both gradients are fp32 sums of exact products (bf16 x bf16 is exact in fp32),
so the fp32 bar of parity.py holds in both types."""
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
    (2, 8, 8, 5, 3, 3, 1, 1, 1),        # one padded quad per row
    (2, 8, 8, 6, 4, 3, 1, 1, 1),        # exactly one quad
    (2, 8, 9, 6, 5, 3, 1, 1, 1),        # one pixel into the next quad; two 32-row tiles
    (1, 8, 16, 3, 128, 3, 1, 1, 1),     # a row fills a chunk
    (1, 16, 8, 3, 129, 3, 1, 1, 1),     # two column segments, the second short
    (1, 4, 16, 2, 301, 3, 1, 1, 1),     # three
    (3, 16, 16, 31, 33, 3, 1, 1, 1),    # one 64 x 64 tile, chunks across images
    (2, 17, 16, 9, 10, 3, 1, 1, 1),     # two tiles, odd channels
    (1, 1, 1, 9, 9, 3, 1, 1, 1),        # rows of 4 reals: half a piece
    (1, 3, 33, 8, 7, 3, 1, 1, 1),       # 12 and 132 reals
    (2, 12, 20, 11, 13, 3, 1, 1, 1),
    (1, 37, 21, 6, 7, 3, 1, 1, 1),      # several tiles each way
    (2, 8, 8, 9, 9, 1, 1, 0, 1),        # 1x1
    (2, 8, 8, 9, 9, 1, 2, 0, 1),        # 1x1 stride 2
    (1, 8, 8, 8, 9, 2, 1, 0, 1),        # two taps
    (1, 8, 8, 9, 9, 4, 1, 1, 1),        # tap groups of 3 and 1
    (1, 8, 8, 11, 9, 5, 2, 2, 1),       # 3 and 2, stride 2
    (1, 7, 8, 15, 15, 7, 2, 3, 1),      # 3, 3 and 1
    (1, 8, 8, 12, 14, 3, 1, 2, 2),      # dilation 2
    (1, 8, 8, 13, 14, 3, 3, 1, 3),      # stride 3, dilation 3
    (1, 16, 16, 70, 2, 3, 1, 1, 1),     # many short rows
    # the four-component kernel's tiles of 32 channels (K steps split over
    # two or four waves)
    (1, 24, 24, 9, 9, 3, 1, 1, 1),
    (1, 32, 64, 9, 9, 3, 2, 1, 1),
    (1, 64, 32, 7, 9, 3, 1, 1, 1),
    (1, 72, 40, 6, 6, 1, 1, 0, 1),
    (3, 32, 32, 13, 11, 3, 1, 1, 1),
    # slices around the reduction's counts of threads (1, 4, 16, eight loads
    # each) in whole and odd runs; dense slices of few and many pixels
    (1, 72, 64, 5, 5, 3, 1, 1, 1),
    (2, 70, 34, 12, 12, 5, 3, 2, 1),
    (4, 40, 24, 28, 28, 1, 1, 0, 1),
    (2, 33, 43, 40, 41, 1, 1, 0, 1),
    (2, 88, 96, 16, 17, 3, 1, 1, 1),
    (1, 66, 40, 14, 15, 5, 1, 2, 1),
    (1, 18, 50, 40, 30, 5, 1, 2, 1),
]


@pytest.mark.parametrize("sep", [False, True], ids=["hamilton", "separable"])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_weight_gradient_rows(shape, dtype, sep):
    say(f"weight gradient rows {dtype} {shape} sep={sep}")
    N, Cin, Cout, H, W, k, s, p, d = shape
    rng = np.random.default_rng(sum(shape) + sep)
    dt = DT[dtype]
    Ho, Wo = quan.conv_out_size(H, k, s, p, d), quan.conv_out_size(W, k, s, p, d)
    x = torch.from_numpy(rng.standard_normal((N, 4, Cin, H, W), dtype=np.float32)).to(dt)
    dy = torch.from_numpy(rng.standard_normal((N, 4, Cout, Ho, Wo), dtype=np.float32)).to(dt)
    w = np.zeros((4, Cout, Cin, k, k))
    fn = quan.quan_qconv2d_separable_backward_weight if sep else quan.quan_qconv2d_backward_weight
    ref_fn = oracle.qconv2d_separable_backward if sep else oracle.qconv2d_backward
    xg, dg = quan.to_device_layout(x.cuda()), quan.to_device_layout(dy.cuda())
    dws, _ = fn(xg, dg, (k, k), stride=s, pad=p, dilation=d, with_bias=False)
    again, _ = fn(xg, dg, (k, k), stride=s, pad=p, dilation=d, with_bias=False)
    torch.cuda.synchronize()
    _, ref, _ = ref_fn(f64(x), w, f64(dy), s, p, d)
    assert_close(np.stack([f64(t) for t in dws]), ref, torch.float32, f"dW {dtype} {shape}")
    assert all(torch.equal(a, b) for a, b in zip(dws, again)), "deterministic"


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_infinite_pixel_stays_out_of_other_taps(dtype):
    """An unpadded 1 x 2 kernel: input column W - 1 meets tap 1 only, and the
    quad of pixels that pads the row would meet it at tap 0.  An infinity
    there must not reach tap 0's gradient."""
    say(f"weight gradient inf {dtype}")
    rng = np.random.default_rng(3)
    x = torch.from_numpy(rng.standard_normal((2, 4, 8, 5, 6), dtype=np.float32)).to(DT[dtype])
    dy = torch.from_numpy(rng.standard_normal((2, 4, 8, 4, 5), dtype=np.float32)).to(DT[dtype])
    _, ref, _ = oracle.qconv2d_backward(f64(x), np.zeros((4, 8, 8, 2, 2)), f64(dy), 1, 0, 1)
    x[..., 5] = float("inf")
    dws, _ = quan.quan_qconv2d_backward_weight(quan.to_device_layout(x.cuda()), quan.to_device_layout(dy.cuda()),
                                               (2, 2), with_bias=False)
    got = np.stack([f64(t) for t in dws])
    assert_close(got[..., 0], ref[..., 0], torch.float32, "tap 0")
    assert not np.isfinite(got[..., 1]).any()


@pytest.mark.parametrize("sep", [False, True], ids=["hamilton", "separable"])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("c,o", [(1, 1), (5, 16), (16, 9), (13, 21)])
def test_component_sum_is_taken_in_fp64(c, o, dtype, sep):
    """Products of component pairs that are exact in fp32 and whose signed sum
    cancels: 2^24 + 1 - 2^24 in eq. 6's and eq. 7's order.  The sum is 1."""
    say(f"weight gradient cancellation {dtype} {c}->{o} sep={sep}")
    dt = DT[dtype]
    x, dy = torch.zeros(1, 4, c, 1, 1), torch.zeros(1, 4, o, 1, 1)
    for q, v in enumerate((4096, 0, 0, 0) if sep else (4096, 1, 4096, 0)):
        x[:, q] = v
    for p, v in enumerate((4096, 2.0 ** -12, -4096, 0) if sep else (4096, 1, -4096, 0)):
        dy[:, p] = v
    fn = quan.quan_qconv2d_separable_backward_weight if sep else quan.quan_qconv2d_backward_weight
    dws, _ = fn(quan.to_device_layout(x.to(dt).cuda()), quan.to_device_layout(dy.to(dt).cuda()), (1, 1), with_bias=False)
    torch.cuda.synchronize()
    assert torch.equal(dws[0].cpu(), torch.ones(o, c, 1, 1))
