"""The stem kernel's bands of output rows: every width of its stored slices
(output channels from 1 to 64), tap counts around a K slice, strides and
dilations, bands of one row, of several and of a whole image, with a short last one, images narrower
than a wave's 32 pixels, and layers whose input rows do not fit LDS; against
the oracle, and the many-row cases against the separate map and convolution
(the same quaternions and products, fp32 sums in another order)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_05512_amd import quan
from parity import assert_close, f64, say

pytestmark = pytest.mark.gpu

BF16 = torch.bfloat16

# (N, H, W, Cout, k, stride, pad, dilation)
SMALL = ([(1, 7, 9, c, 3, 1, 1, 1) for c in (1, 2, 3, 6, 7, 8, 9, 15, 16, 17, 24, 33, 50, 63, 64)] +
         [(2, 9, 37, 16, k, s, k // 2, 1) for k in (1, 2, 4, 5) for s in (1, 2, 3)] +
         [(1, 30, 33, 8, 7, 2, 3, 1), (1, 21, 20, 16, 3, 1, 2, 2), (2, 70, 75, 4, 7, 1, 30, 10),
          (1, 40, 37, 8, 3, 1, 0, 1), (1, 5, 5, 8, 3, 1, 0, 1), (1, 8, 6, 8, 3, 4, 1, 1)] +
         [(n, h, h + 1, c, k, s, k // 2, 1) for n, h, c, k, s in ((5, 14, 36, 3, 1), (3, 37, 64, 1, 2), (2, 26, 64, 3, 1),
                                                                  (2, 43, 24, 5, 2), (1, 69, 24, 5, 1), (1, 33, 16, 7, 1))])
# not staged: 7 rows of 2000 columns; a span of 97 rows
UNSTAGED = [(1, 8, 2000, 8, 7, 2, 3, 1), (1, 101, 99, 4, 7, 1, 48, 16)]
# bands of several rows; odd heights leave a short one
TALL = [(16, 97, 23, 6, 3, 1, 1, 1), (40, 99, 31, 16, 3, 1, 1, 1), (64, 101, 17, 20, 3, 1, 1, 1),
        (64, 203, 45, 16, 3, 2, 1, 1), (64, 37, 37, 64, 1, 2, 0, 1), (64, 27, 27, 38, 3, 2, 1, 1),
        (8, 86, 85, 64, 3, 1, 1, 1), (32, 69, 70, 24, 5, 1, 2, 1), (16, 112, 113, 16, 7, 2, 3, 1)]


def _run(case, scale=1.0):
    N, H, W, Cout, k, s, p, d = case
    rng = np.random.default_rng(sum(case))
    rgb = torch.from_numpy((scale * rng.random((N, 3, H, W), dtype=np.float32))).to(BF16)
    w = torch.from_numpy((rng.standard_normal((4, Cout, 1, k, k)) / np.sqrt(4 * k * k)).astype(np.float32)).to(BF16)
    b = torch.from_numpy((rng.standard_normal((4, Cout)) * 0.1).astype(np.float32)).to(BF16)
    ws = [w[q].contiguous().cuda() for q in range(4)]
    packed, shape = quan.quan_qconv2d_pack_weights(*ws), tuple(ws[0].shape)
    geo = dict(bias=b.cuda(), stride=s, pad=p, dilation=d)
    ho, wo = quan.conv_out_size(H, k, s, p, d), quan.conv_out_size(W, k, s, p, d)
    out = quan.empty_qmap(N, Cout, ho, wo, BF16, torch.device("cuda:0")).fill_(float("nan"))
    quan.quan_qconv2d_poincare_forward(rgb.cuda(), packed, shape, out=out, **geo)
    two = quan.quan_qconv2d_forward_packed(quan.quan_poincare_map(rgb.cuda()), packed, shape, **geo)
    torch.cuda.synchronize()
    return rgb, w, b, out, two


@pytest.mark.parametrize("case", SMALL + UNSTAGED, ids=str)
def test_stem_against_oracle(case):
    say(f"stem {case}")
    rgb, w, b, out, two = _run(case)
    _, _, _, _, _, s, p, d = case
    ref = oracle.qconv2d(oracle.poincare(f64(rgb)), f64(w), f64(b), s, p, d)
    assert_close(f64(out), ref, BF16, f"stem {case}")
    assert_close(f64(out), f64(two), BF16, f"stem vs two passes {case}")


@pytest.mark.parametrize("case", TALL, ids=str)
def test_stem_bands(case):
    say(f"stem bands {case}")
    _, _, _, out, two = _run(case)
    assert_close(f64(out), f64(two), BF16, f"stem vs two passes {case}")


def test_stem_keeps_a_bad_pixel_to_its_windows():
    """An infinite colour makes its own windows NaN and no other output."""
    say("stem infinity")
    rng = np.random.default_rng(1)
    rgb = torch.from_numpy(rng.random((1, 3, 12, 40), dtype=np.float32)).to(BF16)
    rgb[0, 1, 0, 0] = float("inf")
    ws = [torch.from_numpy(rng.standard_normal((8, 1, 3, 3)).astype(np.float32)).to(BF16).cuda() for _ in range(4)]
    out = quan.quan_qconv2d_poincare_forward(rgb.cuda(), quan.quan_qconv2d_pack_weights(*ws), (8, 1, 3, 3), pad=1)
    bad = ~torch.isfinite(out[0].float()).all(0).all(0)
    torch.cuda.synchronize()
    want = torch.zeros(12, 40, dtype=torch.bool)
    want[:2, :2] = True
    assert torch.equal(bad.cpu(), want)
