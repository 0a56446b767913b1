"""The strided input gradient, whose output phases each write their pixels in
place: strides 2 to 4 (up to 16 phases), kernels that leave phases without
taps (zeros), images smaller than the stride, ragged sizes, channel counts
that take the pointwise kernel, the deferred store and the direct one, and
tail blocks, in both forms and types, with dX filled with NaN beforehand.
Against the oracle, and for the large case against fp64 matrix products."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import BF16_ATOL, BF16_RTOL, assert_close, f64, say

pytestmark = pytest.mark.gpu

DT = {"fp32": torch.float32, "bf16": torch.bfloat16}

# (N, Cin, Cout, H, W, k, stride, pad)
SHAPES = [
    (2, 32, 64, 12, 14, 3, 2, 1),     # phases of 1, 2, 2, 4 taps; the first through the pointwise kernel
    (1, 64, 32, 9, 11, 3, 2, 1),
    (1, 64, 64, 13, 10, 3, 2, 0),
    (2, 8, 16, 7, 9, 1, 2, 0),        # three phases without taps
    (1, 8, 16, 10, 11, 2, 3, 0),      # five phases without taps
    (1, 8, 8, 17, 18, 5, 4, 2),       # 16 phases
    (2, 3, 5, 9, 8, 3, 2, 1),         # element-wise everything
    (1, 12, 20, 11, 13, 3, 2, 1),     # partial chunks
    (1, 40, 24, 11, 9, 4, 2, 1),
    (3, 16, 8, 1, 5, 3, 2, 1),        # one row: the odd phases have no pixels
    (1, 96, 8, 6, 6, 3, 3, 1),        # several 64-channel tiles
]


def _case(shape, dt, seed):
    N, Cin, Cout, H, W, k, s, p = shape
    rng = np.random.default_rng(seed)
    ho, wo = quan.conv_out_size(H, k, s, p, 1), quan.conv_out_size(W, k, s, p, 1)
    w = torch.from_numpy((rng.standard_normal((4, Cout, Cin, k, k)) / np.sqrt(4 * Cout * k * k)).astype(np.float32)).to(dt)
    dy = torch.from_numpy(rng.standard_normal((N, 4, Cout, ho, wo)).astype(np.float32)).to(dt)
    return w, dy


def _run(shape, w, dy, sep):
    N, Cin, _, H, W, _, s, p = shape
    dx = quan.empty_qmap(N, Cin, H, W, dy.dtype, torch.device("cuda:0")).fill_(float("nan"))
    fn = quan.quan_qconv2d_separable_backward_data if sep else quan.quan_qconv2d_backward_data
    fn(quan.to_device_layout(dy.cuda()), *[w[q].contiguous().cuda() for q in range(4)], (H, W), stride=s, pad=p, dx=dx)
    torch.cuda.synchronize()
    return dx


@pytest.mark.parametrize("sep", [False, True], ids=["hamilton", "separable"])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_phases_write_in_place(shape, dtype, sep):
    say(f"input gradient by phases {dtype} {shape} sep={sep}")
    N, Cin, _, H, W, _, s, p = shape
    w, dy = _case(shape, DT[dtype], sum(shape))
    ref_fn = oracle.qconv2d_separable_backward if sep else oracle.qconv2d_backward
    ref, _, _ = ref_fn(np.zeros((N, 4, Cin, H, W)), f64(w), f64(dy), s, p, 1)
    assert_close(f64(_run(shape, w, dy, sep)), ref, DT[dtype], f"dX {dtype} {shape}")


def test_phases_with_tail_blocks():
    """36864 pixels a phase and 64 channels: 288 tiles of 128 pixels, so each
    phase ends in claimed 32-pixel blocks on 256 compute units."""
    shape = (4, 64, 64, 192, 192, 3, 2, 1)
    say(f"input gradient by phases, tail blocks {shape}")
    N, Cin, Cout, H, W, k, s, p = shape
    w, dy = _case(shape, torch.bfloat16, 5)
    dx = _run(shape, w, dy, False)
    ho, wo = dy.shape[3:]
    rows = dy.cuda().permute(0, 3, 4, 1, 2).reshape(-1, 4 * Cout).double()
    wd = w.cuda().double()
    ref = torch.zeros((N, H + 2 * p, W + 2 * p, 4 * Cin), dtype=torch.float64, device="cuda")
    neg = {(0, 1), (0, 2), (0, 3), (1, 2), (2, 3), (3, 1)}
    for u in range(k):
        for v in range(k):
            b = torch.stack([torch.stack([(-1.0 if (i, j) in neg else 1.0) * wd[i ^ j, :, :, u, v] for j in range(4)], 1)
                             for i in range(4)])  # [p, o, q, c]
            to = ref[:, u:u + s * (ho - 1) + 1:s, v:v + s * (wo - 1) + 1:s]
            to += (rows @ b.reshape(4 * Cout, 4 * Cin)).reshape(to.shape)
    ref = ref[:, p:p + H, p:p + W].reshape(N, H, W, 4, Cin).permute(0, 3, 4, 1, 2)
    err = (dx.double() - ref).abs()
    assert bool((err <= BF16_ATOL + BF16_RTOL * ref.abs()).all()), float(err.max())
