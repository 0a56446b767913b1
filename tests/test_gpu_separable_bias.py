"""The separable form's bias over several tiles per work-group: 150 pixel tiles
by 1 to 3 channel tiles on 256 compute units, so a work-group's tiles change
their channels between one epilogue and the next; channel counts that end a
tile early, 8- and 16-byte stores.  Against fp64 matrix products."""
import numpy as np
import pytest
import torch

from paper_2509_05512_amd import quan
from parity import BF16_ATOL, BF16_RTOL, say

pytestmark = pytest.mark.gpu

SIGN = ((1, -1, -1, -1), (1, 1, 1, -1), (1, -1, 1, 1), (1, 1, -1, 1))  # eq. 7


@pytest.mark.parametrize("with_bias", [True, False], ids=["bias", "plain"])
@pytest.mark.parametrize("cin", [8, 32])
@pytest.mark.parametrize("cout", [64, 72, 136, 140])
def test_separable_bias_over_tiles(cout, cin, with_bias):
    say(f"separable bias {cin}->{cout} bias={with_bias}")
    n, h, w, k = 8, 48, 50, 3
    rng = np.random.default_rng(cout + cin)
    x = torch.from_numpy(rng.standard_normal((n, 4, cin, h, w), dtype=np.float32)).bfloat16().cuda()
    ws = [torch.from_numpy((rng.standard_normal((cout, cin, k, k)) / np.sqrt(4 * cin * k * k)).astype(np.float32))
          .bfloat16().cuda() for _ in range(4)]
    b = torch.from_numpy((10 * rng.standard_normal((4, cout))).astype(np.float32)).bfloat16().cuda() if with_bias else None
    y = quan.quan_qconv2d_separable_forward(quan.to_device_layout(x), *ws, bias=b, pad=1)
    xp = torch.nn.functional.pad(x.double(), (1, 1, 1, 1))
    c = [sum(xp[:, q, :, u:u + h, v:v + w].permute(0, 2, 3, 1).reshape(-1, cin) @ ws[q][:, :, u, v].double().t().contiguous()
             for u in range(k) for v in range(k)) for q in range(4)]
    for p in range(4):
        ref = sum(SIGN[p][q] * c[q] for q in range(4))
        if with_bias:
            ref = ref + b[p].double()
        ref = ref.reshape(n, h, w, cout).permute(0, 3, 1, 2)
        err = (y[:, p].double() - ref).abs()
        assert bool((err <= BF16_ATOL + BF16_RTOL * ref.abs()).all()), (p, float(err.max()))
